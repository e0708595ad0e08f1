// bf16 GEMM on the gfx950 matrix cores: C[M,N] = A[M,K] * Wt[N,K]^T, fp32 accumulate, fused epilogue.
// Both operands are K-contiguous, so every MFMA operand fragment is one 16-byte LDS read.
//
// Block tile BM x BN x 64, WGM x WGN wavefronts, each owning a (BM/WGM) x (BN/WGN) sub-tile built from
// v_mfma_f32_32x32x16_bf16.  k-tiles go HBM -> LDS directly (no staging registers, no LDS stores) into
// two buffers: k-tile kt+1 is in flight while k-tile kt is multiplied (problems of few tiles take small tiles and a
// ring of loads, see k_gemm_ring and k_gemm_thin; mid-size tiles run in turns, see k_gemm_turns; which takes what: tile_family,
// big_tile, cut_tile).  Operand fragments are
// double-buffered in registers: those of k-step ks+1 are read from LDS while the MFMAs of k-step ks run.
// The issue order of the main loop is pinned (see there): the two wavefronts of a SIMD are served oldest
// first rather than interleaved, so each has to keep the matrix pipe busy on its own; tile loads go out
// one behind an MFMA instead of in a burst, and an MFMA waits only for the LDS reads it needs.
// LDS rows are 128 bytes (64 bf16); LDS serves 16 lanes x 16 bytes per cycle from 64 banks, i.e. two rows per
// bank sweep, so the 16-byte chunk index is XOR-swizzled with (row >> 1) & 7, which spreads a column of
// chunks over all banks.
//
// The epilogue stages the output tile through LDS so that global memory is written (and, for the fp32
// residual update, read) in whole rows, 16 bytes per lane.  EPI_HEADS stores per attention head (q | k | v
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

// The fragments of a k-step are read in the order A row-tile 0, B column-tiles 0 .. TN-1, A row-tiles 1 ..;
// the MFMAs run row-tile by row-tile (n = i * TN + j).  Index of the last fragment MFMA n needs:
template <int TN> constexpr int frag_need(int n) {
  const int i = n / TN, j = n % TN, ia = i == 0 ? 0 : TN + i, ib = 1 + j;
  return ia > ib ? ia : ib;
}
template <int TN> constexpr int frag_need_upto(int n) {
  int m = -1;
  for (int t = 0; t <= n; ++t) m = frag_need<TN>(t) > m ? frag_need<TN>(t) : m;
  return m;
}
// reads k (issued behind MFMA first + k * (NM - first) / NR) that precede MFMA n
template <int NM, int NR> constexpr int reads_before(int n, int first) {
  int c = 0;
  for (int k = 0; k < NR; ++k) c += first + k * (NM - first) / NR < n ? 1 : 0;
  return c;
}
// Accumulators of v_mfma_f32_MF x MF: lane l holds column l % MF and, per register quad q, the four consecutive rows
// q * 8 + (l / MF) * 4 + (0..3)
template <int MF> struct Mfma;
template <> struct Mfma<32> { typedef f32x16 acc; };
template <> struct Mfma<16> { typedef f32x4 acc; };

// A block's epilogue over its BM x BN tile; LB: bytes of LDS (free by now) that it may stage through.
template <int MF, int BM, int BN, int WGM, int WGN, int TM, int TN, int EPI, int LB>
__device__ __forceinline__ void finish_tile(typename Mfma<MF>::acc (&acc)[TM][TN], uint4* smem, int64_t m0, int64_t n0, int64_t M,
                                            int64_t N, int part, int sec, bool swapped, const EpiArgs& e, const HeadsArgs& ha) {
  // The MFMAs ran with the weight rows as the A operand, so a lane holds the output row
  // m = .. + lr and, per register quad q, the four consecutive columns n = .. + q*8 + lg*4 + (0..3).
  // The tile goes through LDS (free now) so that global memory sees whole rows: 16 bytes per lane,
  // consecutive lanes on consecutive addresses.  LDS rows are XOR-swizzled with the row index so that
  // neither the column-wise writes nor the row-wise reads conflict on banks.
  constexpr int NW = WGM * WGN, NT = NW * 64, WM = BM / WGM, WN = BN / WGN, Q = MF == 32 ? 4 : 1;   // register quads of an accumulator tile
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & (MF - 1), lg = lane / MF;
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
    static_assert(BM * BN * 2 <= LB, "EPI_HEADS stages the whole tile at once");
    // [row][wavefront column]: sums of squares; behind the staged tile where there is room
    // Plain sections of 128-column tiles are staged in fp32, so that only the result is rounded, as by the separate kernels
    // (staged in bf16, 64-column tiles left a layer of dim 1664 2.58e-3 from 64 bits, 2.50e-3 this way and by those, in
    // the same time).  The wider tiles' fp32 rows do not all fit.
    constexpr bool WIDE = BN == 128 && BM * BN * 4 + BM * WGN * 4 <= LB;
    constexpr int SB = WIDE ? 4 : 2;
    constexpr bool RED_DYN = BM * BN * SB + BM * WGN * 4 <= LB;
    __shared__ float red_static[RED_DYN ? 1 : BM * WGN];
    float* const red = RED_DYN ? (float*)smem + BM * BN * SB / 4 : red_static;
    const HeadSection sc = ha.sec[sec];
    const int64_t nsec = n0 - (int64_t)sec * ha.dim;     // first column of this tile inside its section
    const int hshift = ha.head_dim == 128 ? 7 : 6, hmask = ha.head_dim - 1;
    uint2* l8 = (uint2*)smem;
    __syncthreads();
    if constexpr (MF == 16) {
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
    }
    if (swapped) {
      // lane: channel row (weight row) nsec + wm*WM + i*32 + lr; register quad: 4 consecutive output rows m
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wm * WM + i * MF + lr;
        const float bvr = bias && n0 + row < N ? bf16_to_f32(bias[n0 + row]) : 0.f;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int nl = wn * WN + j * MF + q * 8 + lg * 4;
            uint2 pk;
            pk.x = cvt_pk_bf16(acc[i][j][q * 4 + 0] + bvr, acc[i][j][q * 4 + 1] + bvr);
            pk.y = cvt_pk_bf16(acc[i][j][q * 4 + 2] + bvr, acc[i][j][q * 4 + 3] + bvr);
            l8[row * UPR + ((nl >> 2) ^ (row & XM))] = pk;
          }
      }
    } else {
      float ss[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) ss[i] = 0.f;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int nl = wn * WN + j * MF + q * 8 + lg * 4;
          float bv[4] = {0.f, 0.f, 0.f, 0.f};
          if (bias && n0 + nl < N) {
            const uint2 b4 = *(const uint2*)(bias + n0 + nl);
            bv[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
            bv[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
          }
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const int row = wm * WM + i * MF + lr;
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              v[t] = acc[i][j][q * 4 + t] + bv[t];
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
        if constexpr (MF == 16) tot += __shfl_xor(tot, 16, 64);
        tot += __shfl_xor(tot, 32, 64);
        if (lg == 0) red[(wm * WM + i * MF + lr) * WGN + wn] = tot;
      }
    }
    __syncthreads();
    if (!swapped && sc.ssq) {
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
    const bool rotate = !swapped && sc.rope, scale = !swapped && (sc.gain || sc.rope);
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
      if (!swapped && sc.gain && col_ok[k]) {
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
            if (WIDE && !swapped) {
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
            if (swapped) {
              const int64_t ch = nsec + row, m = m0 + c8 + k * (BN / 2);   // channel in the section, first of 8 output rows
              if (ch < ha.dim && n0 + row < N && m < M)
                __builtin_nontemporal_store(u32x4{d[g][k].x, d[g][k].y, d[g][k].z, d[g][k].w}, (u32x4*)((bf16_t*)sc.dst + ch * sc.ld + sc.row0 + m));
            } else if (m0 + row < M && col_ok[k]) {
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
  } else if constexpr (EPI != EPI_RESID && EPI != EPI_PART) {
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
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int nl = wn * WN + j * MF + q * 8 + lg * 4;
            float bv[4] = {0.f, 0.f, 0.f, 0.f};
            if (bias && n0 + nl < N) {
              const uint2 b4 = *(const uint2*)(bias + n0 + nl);
              bv[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
              bv[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
              const int row = (SP == 1 ? wm * WM : 0) + i * MF + lr;      // row inside this pass
              float v[4];
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                v[t] = acc[i][j][q * 4 + t] + bv[t];
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
  } else {
    static_assert(MF == 32, "the other accumulators' is in k_gemm_turns");
    // residual stream: x[m, n] += gate[n] * (acc + bias[n]) in fp32 (EPI_PART: this range's x[m, n] = acc).  Passes over the wavefront rows of the
    // block tile and, inside one, over groups of GI 32-row accumulator tiles: as many as fit in LDS as floats
    constexpr int CPR = BN / 4, RPI = 64 / CPR;          // 16-byte chunks (4 floats) per row
    constexpr int GI_FIT = LB / (32 * BN * 4), GI = GI_FIT < TM ? GI_FIT : TM;
    static_assert(GI >= 1, "one 32-row tile of fp32 results must fit the operand buffers");
    float4* l16 = (float4*)smem;
#pragma unroll
    for (int pass = 0; pass < WGM; ++pass) {
#pragma unroll
      for (int i0 = 0; i0 < TM; i0 += GI) {
        const int gi = TM - i0 < GI ? TM - i0 : GI;      // accumulator tiles in this group
        // This wavefront's share of the group's residual rows is requested before the group is staged, so the
        // loads travel while the accumulators go through LDS (same-box A/B at 14400 x 5120 x 5120: 724 -> 679 us)
        constexpr int NIT = (GI * 32 + NW * RPI - 1) / (NW * RPI);
        float4 xpre[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int r = wave * RPI + it * NW * RPI;
          if (r < gi * 32) {
            const int row = r + lane / CPR, p = lane % CPR;
            const int64_t m = m0 + pass * WM + i0 * 32 + row, n = n0 + (p ^ (row & 15)) * 4;
            if (EPI == EPI_RESID && m < M && n < N) xpre[it] = *(const float4*)(e.resid + m * e.ldr + n);
          }
        }
        __syncthreads();
        if (wm == pass) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
              const int nl = wn * WN + j * MF + q * 8 + lg * 4;
              float bv[4] = {0.f, 0.f, 0.f, 0.f};
              float4 gv = make_float4(1.f, 1.f, 1.f, 1.f);
              if (EPI == EPI_RESID && n0 + nl < N) {
                if (bias) {
                  const uint2 b4 = *(const uint2*)(bias + n0 + nl);
                  bv[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
                  bv[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
                }
                if (e.gate) gv = *(const float4*)(e.gate + n0 + nl);
              }
#pragma unroll
              for (int ii = 0; ii < GI; ++ii) {
                if (i0 + ii < TM) {
                  const int row = ii * MF + lr;
                  float4 v;
                  v.x = gv.x * (acc[i0 + ii][j][q * 4 + 0] + bv[0]);
                  v.y = gv.y * (acc[i0 + ii][j][q * 4 + 1] + bv[1]);
                  v.z = gv.z * (acc[i0 + ii][j][q * 4 + 2] + bv[2]);
                  v.w = gv.w * (acc[i0 + ii][j][q * 4 + 3] + bv[3]);
                  l16[row * CPR + ((nl >> 2) ^ (row & 15))] = v;
                }
              }
            }
        }
        __syncthreads();
        // gi * 32 rows, shared out over the wavefronts RPI rows per read; the residual values were requested
        // before the staging above, so they are on their way (or there) by now
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int r = wave * RPI + it * NW * RPI;
          if (r < gi * 32) {
            const int row = r + lane / CPR, p = lane % CPR;
            const float4 v = l16[row * CPR + p];
            const int64_t m = m0 + pass * WM + i0 * 32 + row, n = n0 + (p ^ (row & 15)) * 4;
            if (m < M && n < N) {
              if constexpr (EPI == EPI_PART) {
                *(float4*)(e.resid + (int64_t)part * M * e.ldr + m * e.ldr + n) = v;
                continue;
              }
              float4 xv = xpre[it];
              xv.x += v.x; xv.y += v.y; xv.z += v.z; xv.w += v.w;
              *(float4*)(e.resid + m * e.ldr + n) = xv;
              if (e.out) {
                uint2 pk;
                pk.x = cvt_pk_bf16(xv.x, xv.y);
                pk.y = cvt_pk_bf16(xv.z, xv.w);
                *(uint2*)((bf16_t*)e.out + m * e.ldo + n) = pk;
              }
            }
          }
        }
      }
    }
  }
}

template <int BM, int BN, int WGM, int WGN, int EPI>
__global__ __launch_bounds__(WGM * WGN * 64) void k_gemm_bf16(const bf16_t* __restrict__ A, int64_t lda,
                                                             const bf16_t* __restrict__ Bt, int64_t ldb,
                                                             int64_t M, int64_t N, int64_t K, int tiles_n,
                                                             int tiles, int parts, EpiArgs e, HeadsArgs ha) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int IA = BM * 8 / NT, IB = BN * 8 / NT;      // wavefront load instructions per k-tile (64 chunks each)
  constexpr int STAGE = (BM + BN) * 8;                   // 16-byte chunks per LDS buffer
  static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0, "tile/thread mismatch");
  extern __shared__ uint4 smem[];

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
  const int kt0 = EPI == EPI_PART ? (int)((K / 64) * part / parts) : 0;
  const int KT = EPI == EPI_PART ? (int)((K / 64) * (part + 1) / parts) - kt0 : (int)(K / 64);

  // EPI_HEADS: a tile of a section that is stored channel-major is computed with the operands exchanged
  // (square tiles only), so that its accumulators, staging tile and row stores are those of C^T
  int sec = 0;
  bool swapped = false;
  if constexpr (EPI == EPI_HEADS) {
    sec = (int)(n0 / ha.dim);
    if constexpr (BM == BN) swapped = ha.sec[sec].transposed != 0;
  }
  const bf16_t* const pa = (swapped ? Bt + n0 * ldb : A + m0 * lda) + kt0 * 64;
  const bf16_t* const pb = (swapped ? A + m0 * lda : Bt + n0 * ldb) + kt0 * 64;
  const int64_t lpa = swapped ? ldb : lda, lpb = swapped ? lda : ldb;
  // slot p of a tile holds chunk (p & 7) ^ ((row >> 1) & 7) of row p >> 3; one wavefront instruction
  // fills slots [base, base + 64), lane l the slot base + l
  const bf16_t* gA[IA]; const bf16_t* gB[IB];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int p = (wave * IA + i) * 64 + lane, row = p >> 3, ch = (p & 7) ^ ((row >> 1) & 7);
    gA[i] = pa + row * lpa + ch * 8;
  }
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int p = (wave * IB + i) * 64 + lane, row = p >> 3, ch = (p & 7) ^ ((row >> 1) & 7);
    gB[i] = pb + row * lpb + ch * 8;
  }
  // load instruction q < IA + IB of this wavefront's share of k-tile kt into stage bufi
  auto load_part = [&](int kt, int bufi, int q) __attribute__((always_inline)) {
    if (kt >= KT) return;
    const int t = kt * 64;
    uint4* base = smem + bufi * STAGE;
    if (q < IA) {
      __builtin_amdgcn_global_load_lds((glb_void_t*)(gA[q] + t), (lds_void_t*)(base + (wave * IA + q) * 64), 16, 0, 0);
    } else {
      __builtin_amdgcn_global_load_lds((glb_void_t*)(gB[q - IA] + t), (lds_void_t*)(base + BM * 8 + (wave * IB + q - IA) * 64), 16, 0, 0);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int lr = lane & 31, lg = lane >> 5;
  int arow[TM], brow[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) arow[i] = wm * WM + i * 32 + lr;
#pragma unroll
  for (int j = 0; j < TN; ++j) brow[j] = wn * WN + j * 32 + lr;

  // Software pipeline.  k-tile kt+1 is in flight while k-tile kt is multiplied; the fragments of k-step
  // ks+1 are read while the MFMAs of k-step ks run, one read behind each of the first MFMAs, in the order in
  // which the next step's MFMAs first need them.  The LDS reads are issued through inline assembly and
  // waited for with explicit counts: the compiler would wait for all outstanding reads before the first
  // MFMA of a step (the last of them only two MFMAs old), which stalls a wavefront whenever the other
  // wavefront of its SIMD is not there to fill the gap; here an MFMA waits only for the fragments it
  // needs, issued most of a k-step earlier.  LDS returns reads in order, so "at most c reads outstanding"
  // means every read but the c newest has landed.
  constexpr int NM = TM * TN, NR = TM + TN;              // MFMAs and fragment reads per k-step
  constexpr int NB = NM >= 8 ? 2 : 1;                    // MFMAs of the last k-step issued before the barrier
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  static_assert(WM % 16 == 0 && WN % 16 == 0, "every fragment row of a lane has the same swizzle");
  // chunk (ks * 2 + lg) ^ s of a row, s = (row >> 1) & 7 = (lr >> 1) & 7 for all of this lane's fragment rows,
  // is at byte (ks * 32) ^ swz of the row
  const uint32_t swz = (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;
  uint32_t fbase[NR];                                    // fragment f: LDS byte offset of this lane's row in stage 0
#pragma unroll
  for (int f = 0; f < NR; ++f) {
    const bool is_a = f == 0 || f > TN;
    const int row = is_a ? arow[f == 0 ? 0 : f - TN] : brow[f - 1];
    fbase[f] = lds0 + (uint32_t)((is_a ? 0 : BM * 8) + row * 8) * 16;
  }
  bf16x8 af[2][TM], bfr[2][TN];
  // fragment f of k-step ks of the stage at byte offset `stage` into register buffer `to`
  auto read_frag = [&](uint32_t stage, int ks, int f, int to) __attribute__((always_inline)) {
    const u32x4 v = lds_read16_raw<0>(fbase[f] + (stage + (swz ^ (uint32_t)(ks * 32))));
    if (f == 0) af[to][0] = __builtin_bit_cast(bf16x8, v);
    else if (f <= TN) bfr[to][f - 1] = __builtin_bit_cast(bf16x8, v);
    else af[to][f - TN] = __builtin_bit_cast(bf16x8, v);
  };
  // The NL load instructions of a k-tile are spread, one behind an MFMA, over the NS MFMAs that follow the
  // barrier which frees their stage (the rest of the last k-step and the first k-step of the next k-tile):
  // issued together right behind the barrier they fill the vector-memory queue, and a wavefront that waits
  // there to issue a load cannot issue the MFMAs behind it either.
  constexpr int NL = IA + IB, NS = (NM - NB) + NM;
#pragma unroll
  for (int q = 0; q < NL; ++q) load_part(0, 0, q);
  tile_barrier();
  static_for<NL>([&](auto q_) __attribute__((always_inline)) {
    constexpr int q = decltype(q_)::value;
    if constexpr (q * NS / NL < NM - NB) load_part(1, 1, q);           // the part that k-step 3 would have issued
  });
#pragma unroll
  for (int f = 0; f < NR; ++f) read_frag(0, 0, f, 0);
  for (int kt = 0; kt < KT; ++kt) {
    const int st = kt & 1;                               // stage of this k-tile
    const uint32_t cur = (uint32_t)st * STAGE * 16, nxt = (uint32_t)(st ^ 1) * STAGE * 16;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      static_for<NM>([&](auto n_) __attribute__((always_inline)) {
        constexpr int n = decltype(n_)::value, i = n / TN, j = n % TN;
        constexpr int need = frag_need<TN>(n), prev = n == 0 ? -1 : frag_need_upto<TN>(n - 1);
        if (ks < 3) {
          // reads of step ks+1 issued so far in this step: those with k * NM / NR < n
          if constexpr (need > prev) lds_wait<NR - 1 - need + reads_before<NM, NR>(n, 0)>();
        } else {
          if constexpr (n < NB) { if constexpr (need > prev) lds_wait<NR - 1 - need>(); }
          if constexpr (n == NB) tile_barrier();   // every read of this k-tile has landed (lgkmcnt(0) precedes it)
        }
        __builtin_amdgcn_sched_barrier(0);               // the MFMA stays behind the wait for its fragments
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks & 1][j], af[ks & 1][i], acc[i][j], 0, 0, 0);
        static_for<NR>([&](auto k_) __attribute__((always_inline)) {
          constexpr int k = decltype(k_)::value;
          if (ks < 3) { if constexpr (k * NM / NR == n) read_frag(cur, ks + 1, k, (ks + 1) & 1); }
          else { if constexpr (n >= NB && NB + k * (NM - NB) / NR == n) read_frag(nxt, 0, k, 0); }
        });
        static_for<NL>([&](auto q_) __attribute__((always_inline)) {
          constexpr int q = decltype(q_)::value, slot = q * NS / NL;       // MFMAs after the barrier
          if (ks == 3) { if constexpr (n >= NB && slot == n - NB) load_part(kt + 2, st, q); }
          else if (ks == 0) { if constexpr (slot == (NM - NB) + n) load_part(kt + 1, st ^ 1, q); }
        });
        __builtin_amdgcn_sched_barrier(0);               // keeps the MFMAs, reads, loads and waits in this order
      });
    }
  }
  lds_wait<0>();

  finish_tile<32, BM, BN, WGM, WGN, TM, TN, EPI, (BM + BN) * 256>(acc, smem, m0, n0, M, N, part, sec, swapped, e, ha);
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
  // work ids as in k_gemm_bf16: a contiguous run per XCD, tiles in bands of 4 tile rows
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

// Mid-size tiles: 2 x 4 wavefronts of (TM * 16) x (TN * 16), v_mfma_f32_16x16x32_bf16, k-slabs of KB in a ring of ST LDS stages.
// The two wavefronts of a SIMD (one of each block half) take turns: while one multiplies a slab, the other reads its next
// slab's fragments and issues its share of the tile loads, with a barrier at every change of roles.  Nothing is interleaved
// by hand and a wavefront needs no second fragment buffer; ST - 1 slabs are in flight, waited for by count.
// What bounds it: LDS.  A slab of 160 x 256 x 64 takes 1280 matrix-pipe cycles per SIMD and 147 KB of fragment reads (1150
// cycles at 128 bytes a cycle) plus 53 KB of tile writes.  Five 16-row tiles by four use 18 reads per 40 MFMAs where one column
// of five 32-row tiles took 24 per 20.  Measured against that layout (one block column per wavefront, pinned order, three
// stages; plain store, us): 6240 x 1536 x 8960 173 -> 155, 6240 x 1536 x 1536 33.9 -> 31.2, 1560 x 4608 x 1536 as 128 x 256
// tiles 30.2 -> 25.0; against a ring of four stages without turns 1008 x 4096 x 1024 (128 x 128) 15.5 -> 11.8.  Counted at 6240 x 1536 x
// 8960 with the residual epilogue: matrix pipes busy 50 % of the cycles at 2.12 GHz, 57 % of those in which a CU has a block, where
// that layout was busy 50 % at 1.93 GHz: what the saved LDS reads gave is clock.
template <int TM, int TN, int KB, int ST, int EPI>
__global__ __launch_bounds__(512) void k_gemm_turns(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ Bt,
                                                   int64_t ldb, int64_t M, int64_t N, int64_t K, int tiles_n, int tiles,
                                                   int parts, EpiArgs e, HeadsArgs ha) {
  constexpr int WGM = 2, WGN = 4, NT = 512;
  constexpr int WM = TM * 16, WN = TN * 16, BM = WGM * WM, BN = WGN * WN;
  constexpr int CPR = KB / 8;                            // 16-byte chunks of an LDS row
  constexpr int ACH = BM * CPR, BCH = BN * CPR, STAGE = ACH + BCH;
  constexpr int IA = (ACH + NT - 1) / NT, IB = BCH / NT, NL = IA + IB;   // load instructions per wavefront and slab
  constexpr bool RAG = ACH % NT != 0;                    // the last wavefronts have one A load less
  constexpr int KS = KB / 32, D = ST - 1;                // k-steps of a slab, slabs in flight
  static_assert(BCH % NT == 0 && ACH % 64 == 0 && (KB == 32 || KB == 64), "whole wavefront instructions");
  extern __shared__ uint4 smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  // work ids as in k_gemm_bf16: a contiguous run per XCD, tiles in bands of 4 tile rows
  const int pid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (pid >= tiles * parts) return;
  const int part = EPI == EPI_PART ? pid / tiles : 0, tile = EPI == EPI_PART ? pid % tiles : pid;
  const int tiles_m = tiles / tiles_n;
  const int band = tile / (4 * tiles_n), in_band = tile % (4 * tiles_n);
  const int band_rows = tiles_m - band * 4 < 4 ? tiles_m - band * 4 : 4;
  const int64_t m0 = (int64_t)(band * 4 + in_band % band_rows) * BM, n0 = (int64_t)(in_band / band_rows) * BN;
  const int s0 = EPI == EPI_PART ? (int)((K / KB) * part / parts) : 0;
  const int NS = EPI == EPI_PART ? (int)((K / KB) * (part + 1) / parts) - s0 : (int)(K / KB);

  // Slot p of a slab holds chunk (p % CPR) ^ swz(row) of row p / CPR, swz spreading a column of chunks over the banks (two
  // 128-byte rows or four 64-byte rows make one sweep of the 64 banks).  Rows beyond the matrix read as zeros.
  auto swz = [](int row) __attribute__((always_inline)) { return CPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };
  const bf16_t* const pa = A + m0 * lda + s0 * KB;
  const bf16_t* const pb = Bt + n0 * ldb + s0 * KB;
  const int64_t left_a = ((M - m0) * lda - s0 * KB) * 2, left_b = ((N - n0) * ldb - s0 * KB) * 2;
  const uint32_t na = (uint32_t)(left_a < 0x7fffffff ? left_a : 0x7fffffff), nb = (uint32_t)(left_b < 0x7fffffff ? left_b : 0x7fffffff);
  uint32_t va[IA], vb[IB];
#pragma unroll
  for (int q = 0; q < IA; ++q) { const int p = (q * 8 + wave) * 64 + lane, row = p / CPR; va[q] = (uint32_t)(row * lda + ((p % CPR) ^ swz(row)) * 8) * 2; }
#pragma unroll
  for (int q = 0; q < IB; ++q) { const int p = (q * 8 + wave) * 64 + lane, row = p / CPR; vb[q] = (uint32_t)(row * ldb + ((p % CPR) ^ swz(row)) * 8) * 2; }
  auto load_slab = [&](int s, int st) __attribute__((always_inline)) {
    uint4* const base = smem + st * STAGE;
#pragma unroll
    for (int q = 0; q < IA; ++q)
      if (!RAG || (q * 8 + wave) * 64 < ACH) load_lds16(pa, na, va[q], s * KB * 2, base + (q * 8 + wave) * 64);
#pragma unroll
    for (int q = 0; q < IB; ++q) load_lds16(pb, nb, vb[q], s * KB * 2, base + ACH + (q * 8 + wave) * 64);
  };
  // at most d slabs of this wavefront's loads outstanding
  const bool all_a = !RAG || ((IA - 1) * 8 + wave) * 64 < ACH;
  auto wait_slabs = [&](auto d_) __attribute__((always_inline)) {
    constexpr int d = decltype(d_)::value;
    if (all_a) vm_wait<d * NL>(); else vm_wait<d * (NL - 1)>();
  };
  auto wait_behind = [&](int behind) __attribute__((always_inline)) {    // slabs issued behind the one waited for
    static_for<D>([&](auto d_) __attribute__((always_inline)) {
      constexpr int d = decltype(d_)::value;
      if (d == D - 1 ? behind >= d : behind == d) wait_slabs(d_);
    });
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
  const uint32_t fa = lds0 + (uint32_t)((wm * WM + lr) * CPR) * 16, fb = lds0 + (uint32_t)(ACH + (wn * WN + lr) * CPR) * 16;
  const uint32_t sx = (uint32_t)(lg ^ swz(lr)) * 16;     // a lane's rows are 16 apart: one swizzle for all of them

  // EPI_RESID: the tile is staged and updated in steps of GI accumulator rows of both block halves, the fp32 residual rows in
  // whole rows, 16 bytes per lane.  The first step's are requested with the last slab's fragments, when no tile loads are left
  // to wait for, and travel while that slab is multiplied; the second step's follow behind the multiplication.
  constexpr bool FP32 = EPI == EPI_RESID || EPI == EPI_PART;
  constexpr int NG = BM * BN * 4 <= STAGE * ST * 16 ? 1 : 2, GI = (TM + NG - 1) / NG;
  static_assert(!FP32 || 2 * GI * 16 * BN * 4 <= STAGE * ST * 16, "a step fits");
  constexpr int CPF = BN / 4, RPW = 64 / CPF, NX = 2 * GI * 16 / 8 / RPW;          // 16-byte chunks per row, rows per read, reads per step
  float4 xv[EPI == EPI_RESID ? NG : 1][EPI == EPI_RESID ? NX : 1];
  // row and first column, inside the tile, of this lane's chunk of read t of step g, and its place in LDS
  auto fp32_at = [&](int g, int t, int& row, int& col, int& at) __attribute__((always_inline)) {
    const int gi = TM - g * GI < GI ? TM - g * GI : GI;   // accumulator rows of this step
    const int r = (t * 8 + wave) * RPW + lane / CPF, half = r / (gi * 16), p = lane % CPF;
    row = half * WM + g * GI * 16 + r % (gi * 16);
    col = (p ^ (r & 15)) * 4;
    at = r * CPF + p;
    return r < 2 * gi * 16;
  };
  auto resid_load = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NX; ++t) {
      int row, col, at;
      if (fp32_at(g, t, row, col, at) && m0 + row < M && n0 + col < N) xv[g][t] = *(const float4*)(e.resid + (m0 + row) * e.ldr + n0 + col);
    }
  };

#pragma unroll
  for (int z = 0; z < D; ++z) if (z < NS) load_slab(z, z);
  wait_behind(NS - 1);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  if (wm == 1) __builtin_amdgcn_s_barrier();             // the second half starts half a slab later
  __builtin_amdgcn_sched_barrier(0);
  // EXCH: operands exchanged, the accumulators are those of C^T
  auto multiply = [&](auto exch_) __attribute__((always_inline)) {
    constexpr bool EXCH = decltype(exch_)::value;
    int cur = 0, prev = ST - 1;
    bf16x8 af[KS][TM], bfr[KS][TN];
    auto slab = [&](int s, auto last_) __attribute__((always_inline)) {
      constexpr bool LAST = decltype(last_)::value;
      const uint32_t base = (uint32_t)cur * STAGE * 16;
      __builtin_amdgcn_sched_barrier(0);
      static_for<KS>([&](auto k_) __attribute__((always_inline)) {
        constexpr int k = decltype(k_)::value;
        const uint32_t o = base + (sx ^ (uint32_t)(k * 64));
        static_for<TN>([&](auto j_) __attribute__((always_inline)) { constexpr int j = decltype(j_)::value; bfr[k][j] = __builtin_bit_cast(bf16x8, lds_read16_raw<j * 256 * CPR>(fb + o)); });
        static_for<TM>([&](auto i_) __attribute__((always_inline)) { constexpr int i = decltype(i_)::value; af[k][i] = __builtin_bit_cast(bf16x8, lds_read16_raw<i * 256 * CPR>(fa + o)); });
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!LAST) {
        // into the stage of slab s - 1, which everyone has read: its reads were waited for before the last barrier
        if (s + D < NS) load_slab(s + D, prev);
        wait_behind(NS - 2 - s < D - 1 ? NS - 2 - s : D - 1);            // slab s + 1 has landed
      } else if constexpr (EPI == EPI_RESID) {
        resid_load(0);
      }
      lds_wait<0>();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
      static_for<KS>([&](auto k_) __attribute__((always_inline)) {
        constexpr int k = decltype(k_)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = EXCH ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[k][i], bfr[k][j], acc[i][j], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[k][j], af[k][i], acc[i][j], 0, 0, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
      if constexpr (!LAST) { __builtin_amdgcn_s_barrier(); __builtin_amdgcn_sched_barrier(0); }
      prev = cur; cur = cur + 1 == ST ? 0 : cur + 1;
    };
    for (int s = 0; s < NS - 1; ++s) slab(s, std::false_type{});
    slab(NS - 1, std::true_type{});
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
  if constexpr (FP32) {
    const bf16_t* bias = (const bf16_t*)e.bias;
    float4* l16 = (float4*)smem;
    static_for<NG>([&](auto g_) __attribute__((always_inline)) {
      constexpr int g = decltype(g_)::value, gi = TM - g * GI < GI ? TM - g * GI : GI;
      if constexpr (EPI == EPI_RESID && g + 1 < NG) resid_load(g + 1);
      __syncthreads();                                   // the operand slabs / the previous step are done with
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int nl = wn * WN + j * 16 + lg * 4;
        float bv[4] = {0.f, 0.f, 0.f, 0.f};
        float4 gv = make_float4(1.f, 1.f, 1.f, 1.f);
        if (EPI == EPI_RESID && n0 + nl < N) {
          if (bias) {
            const uint2 b4 = *(const uint2*)(bias + n0 + nl);
            bv[0] = bf16_to_f32((bf16_t)(b4.x & 0xffff)); bv[1] = bf16_to_f32((bf16_t)(b4.x >> 16));
            bv[2] = bf16_to_f32((bf16_t)(b4.y & 0xffff)); bv[3] = bf16_to_f32((bf16_t)(b4.y >> 16));
          }
          if (e.gate) gv = *(const float4*)(e.gate + n0 + nl);
        }
#pragma unroll
        for (int i = 0; i < gi; ++i) {
          const f32x4 a = acc[g * GI + i][j];
          const int r = (wm * gi + i) * 16 + lr;
          l16[r * CPF + ((nl >> 2) ^ (r & 15))] = make_float4(gv.x * (a[0] + bv[0]), gv.y * (a[1] + bv[1]), gv.z * (a[2] + bv[2]), gv.w * (a[3] + bv[3]));
        }
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NX; ++t) {
        int row, col, at;
        if (!fp32_at(g, t, row, col, at)) continue;
        const float4 v = l16[at];
        const int64_t m = m0 + row, n = n0 + col;
        if (m >= M || n >= N) continue;
        if constexpr (EPI == EPI_PART) {
          *(float4*)(e.resid + ((int64_t)part * M + m) * e.ldr + n) = v;
        } else {
          float4 x = xv[g][t];
          x.x += v.x; x.y += v.y; x.z += v.z; x.w += v.w;
          *(float4*)(e.resid + m * e.ldr + n) = x;
          if (e.out) *(uint2*)((bf16_t*)e.out + m * e.ldo + n) = make_uint2(cvt_pk_bf16(x.x, x.y), cvt_pk_bf16(x.z, x.w));
        }
      }
    });
  } else {
    finish_tile<16, BM, BN, WGM, WGN, TM, TN, EPI, STAGE * ST * 16>(acc, smem, m0, n0, M, N, part, sec, exch, e, ha);
  }
}

template <int TM, int TN, int KB, int ST, int EPI>
static void launch_turns(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N,
                         int64_t K, const EpiArgs& e, hipStream_t st, int parts) {
  constexpr int BM = 32 * TM, BN = 64 * TN;
  constexpr int lds = (BM + BN) * KB * 2 * ST;
  const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN);
  static std::atomic<uint64_t> done;
  allow_dynamic_lds((const void*)k_gemm_turns<TM, TN, KB, ST, EPI>, lds, done);
  HeadsArgs ha{};
  if (EPI == EPI_HEADS) { e.heads->ssq_np = e.heads->dim / BN; ha = *e.heads; }
  dim3 grid((unsigned)((tm * tn * parts + 7) / 8 * 8));
  k_gemm_turns<TM, TN, KB, ST, EPI><<<grid, 512, lds, st>>>(A, lda, Wt, ldw, M, N, K, tn, tm * tn, parts, e, ha);
}
template <int TM, int TN, int KB, int ST>
static bool launch_turns_cfg(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N,
                             int64_t K, int epi, const EpiArgs& e, hipStream_t st, int parts) {
  if (epi == EPI_STORE) launch_turns<TM, TN, KB, ST, EPI_STORE>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_GELU) launch_turns<TM, TN, KB, ST, EPI_GELU>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_RESID) launch_turns<TM, TN, KB, ST, EPI_RESID>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_HEADS) launch_turns<TM, TN, KB, ST, EPI_HEADS>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else if (epi == EPI_PART) launch_turns<TM, TN, KB, ST, EPI_PART>(A, lda, Wt, ldw, M, N, K, e, st, parts);
  else return false;
  return true;
}

template <int BM, int BN, int WGM, int WGN, int EPI>
static void launch_one(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N,
                       int64_t K, const EpiArgs& e, hipStream_t st, int parts = 1) {
  constexpr int NT = WGM * WGN * 64;
  constexpr size_t lds = (size_t)(BM + BN) * 256;        // two k-tiles
  const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN);
  static std::atomic<uint64_t> done;
  allow_dynamic_lds((const void*)k_gemm_bf16<BM, BN, WGM, WGN, EPI>, (int)lds, done);
  HeadsArgs ha{};
  if (EPI == EPI_HEADS) { e.heads->ssq_np = e.heads->dim / BN; ha = *e.heads; }
  dim3 grid((unsigned)((tm * tn * parts + 7) / 8 * 8));
  k_gemm_bf16<BM, BN, WGM, WGN, EPI><<<grid, NT, lds, st>>>(A, lda, Wt, ldw, M, N, K, tn, tm * tn, parts, e, ha);
}
// false: this tile shape has no such epilogue (the rules below never ask for it)
template <int BM, int BN, int WGM, int WGN>
static bool launch_cfg(const bf16_t* A, int64_t lda, const bf16_t* Wt, int64_t ldw, int64_t M, int64_t N,
                       int64_t K, int epi, const EpiArgs& e, hipStream_t st, int parts) {
  constexpr bool HEADS = BM == 256, PART = BM == 256;
  if (epi == EPI_STORE) launch_one<BM, BN, WGM, WGN, EPI_STORE>(A, lda, Wt, ldw, M, N, K, e, st);
  else if (epi == EPI_GELU) launch_one<BM, BN, WGM, WGN, EPI_GELU>(A, lda, Wt, ldw, M, N, K, e, st);
  else if (epi == EPI_RESID) launch_one<BM, BN, WGM, WGN, EPI_RESID>(A, lda, Wt, ldw, M, N, K, e, st);
  else if (epi == EPI_HEADS && HEADS) { if constexpr (HEADS) launch_one<BM, BN, WGM, WGN, EPI_HEADS>(A, lda, Wt, ldw, M, N, K, e, st); }
  else if (epi == EPI_PART && PART) { if constexpr (PART) launch_one<BM, BN, WGM, WGN, EPI_PART>(A, lda, Wt, ldw, M, N, K, e, st, parts); }
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
// x[m, n] += gate[n] * (bias[n] + sum over the K ranges, in range order), and its rounded copy
__global__ __launch_bounds__(256) void k_add_parts(const float* __restrict__ part, int parts, int64_t M, int64_t N, EpiArgs e) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= M * N) return;
  const int64_t m = i / N, n = i % N;
  float4 s = *(const float4*)(part + i);
  for (int p = 1; p < parts; ++p) {
    const float4 v = *(const float4*)(part + (int64_t)p * M * N + i);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  if (e.bias) {
    const uint2 b = *(const uint2*)((const bf16_t*)e.bias + n);
    s.x += bf16_to_f32((bf16_t)(b.x & 0xffff)); s.y += bf16_to_f32((bf16_t)(b.x >> 16));
    s.z += bf16_to_f32((bf16_t)(b.y & 0xffff)); s.w += bf16_to_f32((bf16_t)(b.y >> 16));
  }
  float4 x = *(const float4*)(e.resid + m * e.ldr + n);
  const float4 g = e.gate ? *(const float4*)(e.gate + n) : make_float4(1.f, 1.f, 1.f, 1.f);
  x.x += g.x * s.x; x.y += g.y * s.y; x.z += g.z * s.z; x.w += g.w * s.w;
  *(float4*)(e.resid + m * e.ldr + n) = x;
  if (e.out) *(uint2*)((bf16_t*)e.out + m * e.ldo + n) = make_uint2(cvt_pk_bf16(x.x, x.y), cvt_pk_bf16(x.z, x.w));
}
size_t gemm_bf16_scratch_bytes(int64_t M, int64_t N) {
  const size_t most = (size_t)256 * 256 * 256 * 4, need = (size_t)(8 * M * N * 4);      // one round of 256 x 256 tiles
  return need < most ? need : most;
}
// Cutting K.  A long K over few tiles leaves most CUs idle, and small tiles in the hundreds move several times the bytes of
// large ones through the caches.  Tiles whose K is cut over blocks until about one round of CUs is full do neither, for the
// price of one fp32 partial result per range, written and read once.  Costs in us per launch, from measurement: a k-tile of a
// block 0.5 (128 x 128), 0.75 (128 x 256), 0.9 (160 x 256), 1.3 (256 x 256), 0.27 for each 64 x 64 block on the CU; 7 for both
// launches and a block's ends, partials at 6.5 TB/s; uncut 0.185 per k-tile and 3.3 (32 x 64), 0.24 per k-tile and 64 x 64 block
// on the CU and 5, 9 (128 x 128) or 14 for launch and ends.  Cut / best uncut in us: 500 x 1536 x 8960 27.9 (128 x 128, 5 ranges) / 43, 1560 x 1536 x 8960 55 (128 x 256,
// 3) / 77, 1008 x 2048 x 8192 45 (128 x 256, 4) / 64, 2560 x 2048 x 8192 88 (160 x 256, 2) / 104, 480 x 3584 x 19456 83 (160 x 256, 6)
// / 158; left uncut 1288 x 5120 x 13824 180 (cut 204), 3000 x 1024 x 4096 41 (42).  Outputs narrower than 768 columns
// are left on the 64-, 160- and 256-row tiles and on the figures of an earlier measurement (a k-tile 1.25 at 160
// rows, 8 for ends and 3 for the second launch, 4 TB/s).  That line is no property of the tiles: the 128-row ones have not been
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
    const double kt = u.bm == 128 ? 0.75 : u.bm == 160 ? 0.9 : u.bm == 192 ? 1.15 : u.bm == 256 ? 1.3 : 1.6;
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
        {fits160 && t160 * p <= 256 && deep ? (narrow ? 1.25 : 0.9) * kt + big : 1e30, {160, 256, 3, p}},
        {!narrow && tiles(128, 256) * p <= 256 && deep ? 0.75 * kt + big : 1e30, {128, 256, 3, p}},
        {!narrow && tiles(128, 128) * p <= 256 && deep ? 0.5 * kt + big : 1e30, {128, 128, 4, p}},
        {t64 * p <= 512 && KT / p >= 4 ? 0.27 * kt * (double)((t64 * p + 255) / 256) + small : 1e30, {64, 64, 4, p}}};
    for (const auto& o : opt)
      if (o.c < best) { best = o.c; r = o.t; }
  }
  return r;
}

// One block per CU at a time, so a launch costs ceil(blocks / 256) rounds of one block's duration.  Durations over that of a
// 256 x 256 block, from whole rounds of blocks at K = 1536 ... 13824, each tile forced in turn: 320 rows 1.15 ... 1.25, 192 rows
// 0.81 ... 0.88, and in turns 160 rows 0.62 ... 0.69 (the fp32 epilogue, whose reads are ahead of it, at the lower end), 128 rows
// 0.53 ... 0.59.  Where they decide (us): 1560 x 4608 x 1536 128 rows, one round, 29, 160 rows 33, 256 rows 42; 2500 x 3072 x
// 12288 168, 182, 254; 3600 x 13824 x 5120 160 rows in 5 rounds 437, 320 rows in 3 454; 18720 x 1536 x 8960 160 rows in 3 467, 256
// rows in 2 488; 7800 x 4608 x 1536 160 rows in 4 117, 256 rows in 3 122; 14400 x 15360 x 5120 256 rows in 14 1850, 128 rows in
// 27 1931; 14400 x 13824 x 5120 320 rows in 10 1601, 160 rows in 19 1634.
// The 192- and 320-row tiles read rows beyond M up to their own multiple, so they are used only where that stays inside the
// 256-row padding the caller guarantees.  The tiles that run in turns read nothing beyond M.  Narrow outputs and plain stores
// take them only where they fit the padding too (160 rows) or nearly fill the round (128 rows).  Those lines are no property of the
// tiles either: beyond them the tiles in turns have not been measured, and the parity tests of the 192- and 256-row tiles
// are such shapes.
static GemmRoute big_tile(int64_t M, int64_t N, int epi) {
  const int64_t tn = (N + 255) / 256, mpad = (M + 255) / 256 * 256;
  const bool heads = epi == EPI_HEADS, any = heads || (epi == EPI_RESID && N >= 1536) || (epi == EPI_GELU && N >= 2048);
  auto tiles = [&](int64_t rows) { return (M + rows - 1) / rows * tn; };
  auto fits = [&](int64_t rows) { return (M + rows - 1) / rows * rows <= mpad; };
  auto cost = [&](int64_t rows, double duration, bool ok) { return ok ? duration * (double)((tiles(rows) + 255) / 256) : 1e30; };
  const GemmRoute tile[5] = {{320, 256, 2, 1}, {256, 256, 2, 1}, {160, 256, 3, 1}, {192, 256, 2, 1}, {128, 256, 3, 1}};
  const double c[5] = {cost(320, 1.23, !heads && fits(320)), cost(256, 1.0, true), cost(160, epi == EPI_RESID ? 0.66 : 0.69, any || fits(160)),
                       cost(192, 0.88, !heads && fits(192)), cost(128, 0.57, any || (tiles(128) > 210 && tiles(128) <= 256))};
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
#define GEMM_TILE(BM, BN, WGM, WGN) \
  if (r.bm == BM) ok = launch_cfg<BM, BN, WGM, WGN>(A, lda, Wt, ldw, M, N, K, ep, ea, st, r.parts)
#define TURNS_TILE(TM, TN, KB, ST) \
  if (r.bm == 32 * TM && r.bn == 64 * TN && r.stages == ST) ok = launch_turns_cfg<TM, TN, KB, ST>(A, lda, Wt, ldw, M, N, K, ep, ea, st, r.parts)
  if (r.bm == 32) ok = launch_thin_cfg(A, lda, Wt, ldw, M, N, K, ep, ea, st);
  else RING_TILE(4);
  else RING_TILE(3);
  else TURNS_TILE(4, 2, 64, 4);
  else TURNS_TILE(4, 4, 64, 3);
  else TURNS_TILE(5, 4, 64, 3);
  else GEMM_TILE(192, 256, 2, 4);
  else GEMM_TILE(256, 256, 2, 4);
  else GEMM_TILE(320, 256, 2, 4);
#undef RING_TILE
#undef GEMM_TILE
#undef TURNS_TILE
  if (r.parts > 1) k_add_parts<<<(unsigned)((M * N / 4 + 255) / 256), 256, 0, st>>>(e.scratch, r.parts, M, N, e);
  return ok;
}
