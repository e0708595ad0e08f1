// Flash attention on the gfx950 matrix cores for the DP_BF16 path: the block's queries attend over one
// contiguous key range [cached prefix ; current block] streamed from HBM through LDS tiles, with an
// online softmax in fp32.  Used for self-attention (cache + block) and cross-attention (text keys).
//
// Scores are computed transposed, S^T = K * Q^T (keys are MFMA rows, queries MFMA columns): a lane
// then owns one query column, so the softmax maximum and sum are reductions over the lane's own
// registers plus one exchange with lane ^ 32, and the fp32 S^T accumulators, once exponentiated and
// rounded to bf16, ARE the B operand of the second product O^T = V^T * P^T.  The rows of a K tile are
// stored in a permuted order so that the eight accumulators a lane packs into one operand belong to
// eight consecutive keys, which makes the matching V^T operand one plain 16-byte LDS read.
//
// Q arrives pre-multiplied by log2(e)/sqrt(head_dim), so scores are base-2 logits.  The softmax reference
// m of a query is folded into the accumulator that the score MFMAs start from (-m instead of 0), so the
// matrix cores hand back s - m and the vector unit only has to exponentiate.  Fast pass: m is fixed once,
// to the query's maximum over the first 32 keys of the tile it starts with, and never raised, so O^T needs no
// rescaling and the loop body is straight-line code.  This is exact as long as nothing overflows: P (bf16)
// and the fp32 sums have 8 exponent bits, so scores may exceed m by ~2^100 before anything is lost.  A
// block whose row sums end up beyond 2^100 (or non-finite) is recomputed by the safe pass, the classical
// online softmax that raises m whenever a tile exceeds it and rescales O^T.
//
// Kernels (attn_bf16_route and attn_bf16_turns have the lines between them).  k_attn_turns: many keys, self- and cross-attention; a
// block of eight wavefronts, the two of a SIMD taking turns at the matrix products and at the exponentials (heads of 128).  k_attn_bf16: fewer keys,
// and heads of 64; its wavefronts are served oldest first rather than interleaved, so its fast pass pins its
// issue order so that one wavefront alone keeps the matrix pipe busy: exponentials between MFMAs, operand fragments read from LDS
// several MFMAs ahead with exact waits (see pass_fast).  Both: 256 queries a block, or 128 with the keys split over two groups of four
// wavefronts, which halves the length of a block; k_attn_bf16 also four wavefronts and 128 queries, two blocks to a CU.  k_attn_few:
// what is small.  Tiles hold 64 keys (k_attn_few 32) and are loaded HBM -> LDS directly.
//
// Grid: one block of 8 wavefronts fits per compute unit, so a grid of them runs in rounds of 256 blocks (512 of 4 wavefronts).  The work ids that
// would make up a last, partly filled round are instead cut into several key ranges each, one block per
// range, which write unnormalised partial results (m, l, O) to a scratch buffer; k_attn_merge joins them.
#include <type_traits>

#include "kernels.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t cvt_pk_bf16(float a, float b) {
  f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// acc + lo + hi of a packed bf16 pair
__device__ __forceinline__ float add_pk_bf16(uint32_t pk, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), __builtin_bit_cast(bf16x2, 0x3f803f80u), acc, false);
}
// LDS has 64 four-byte banks: 16 lanes x 16 bytes are served per cycle.  XOR-swizzling the 16-byte chunk
// index with the row spreads a column of chunks over all banks: rows of 256 bytes use row & 15, rows of
// 128 bytes (two rows per bank sweep) use (row >> 1) & 7.
template <int CR> __device__ __forceinline__ int kswz(int row) { return CR == 16 ? (row & 15) : ((row >> 1) & 7); }
// tile row -> key held in that row: bits 2 and 3 of the row index are exchanged
__device__ __forceinline__ int swap23(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

template <int OFF> __device__ __forceinline__ bf16x8 lds_read16(uint32_t addr) {
  return __builtin_bit_cast(bf16x8, lds_read16_raw<OFF>(addr));
}

// Deferred RMSNorm of the queries: a row's sum of squares arrives as qn.np partial sums; lanes of parity 0 and 1 add up the even and
// the odd ones, in order.  The first PS of a lane are requested before anything else, so that they and what is requested behind
// them are one trip to memory and none waits for what comes later; more of them (wide models on 64-column tiles) are read PS at a
// time when they are added up (480 queries x 75 keys x 28 heads of 128, 56 partial sums, in a stage: one at a time 15.9 us, 13.0 this way).
struct QuerySums {
  static constexpr int PS = 12;
  float v[PS];
  const float* p;
  __device__ __forceinline__ void request(const AttnQNorm& qn, int64_t row, int64_t S, int parity) {
    p = qn.ssq + (row < S ? row : S - 1);
    if (!qn.ssq) return;
    static_for<PS / 4>([&](auto g_) __attribute__((always_inline)) {
      constexpr int g = decltype(g_)::value * 4;
#pragma unroll
      for (int u = g; u < g + 4; ++u) v[u] = 0.f;
      if (2 * g < qn.np) {                               // no loads that few sums do not need: every wavefront of a block makes them
#pragma unroll
        for (int u = g; u < g + 4; ++u) v[u] = p[(parity + 2 * u < qn.np ? parity + 2 * u : 0) * qn.stride];
      }
    });
  }
  // the factor of the row; O: distance to a lane of the other parity
  template <int O> __device__ __forceinline__ float factor(const AttnQNorm& qn, int parity) const {
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < PS; ++u) sum += parity + 2 * u < qn.np ? v[u] : 0.f;
    for (int i0 = parity + 2 * PS; i0 < qn.np; i0 += 2 * PS) {
      float w[PS];
#pragma unroll
      for (int u = 0; u < PS; ++u) w[u] = p[(i0 + 2 * u < qn.np ? i0 + 2 * u : 0) * qn.stride];
#pragma unroll
      for (int u = 0; u < PS; ++u) sum += i0 + 2 * u < qn.np ? w[u] : 0.f;
    }
    sum += __shfl_xor(sum, O, 64);
    return rsqrtf(sum * qn.inv_dim + qn.eps) * qn.scale;
  }
};
template <int KS> __device__ __forceinline__ void scale_queries(bf16x8 (&qf)[KS], float r) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[ks][e] = (__bf16)((float)qf[ks][e] * r);
}
// The fragments of 32 queries from row q0 of a head: B operand, column = query lr, 8 head-dim values per lane
template <int KS, int HD>
__device__ __forceinline__ void request_queries(const bf16_t* __restrict__ qh, int64_t q0, int lr, int lg, int64_t S, const AttnQNorm& qn,
                                                QuerySums& qs, bf16x8 (&qf)[KS]) {
  qs.request(qn, q0 + lr, S, lg);
  qh += (q0 + lr) * HD + lg * 8;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, *(const uint4*)(qh + ks * 16));
  __builtin_amdgcn_sched_barrier(0);
}

template <int HD, int QG, int KG>
__global__ __launch_bounds__(QG * KG * 64, 2) void k_attn_bf16(const bf16_t* __restrict__ q, int64_t q_head_stride,
                                                  const bf16_t* __restrict__ k, int64_t k_head_stride,
                                                  int64_t k_row0, const bf16_t* __restrict__ vt,
                                                  int64_t vt_row_stride, int64_t S, int64_t L,
                                                  bf16_t* __restrict__ out, int64_t ldo, int qblocks,
                                                  int n_full, int n_tail, int parts,
                                                  float* __restrict__ partial, AttnQNorm qn) {
  constexpr int CR = HD / 8;                 // 16-byte chunks per K row
  constexpr int KS = HD / 16;                // MFMA k-steps over the head dim
  constexpr int DT = HD / 32;                // 32-row tiles of O^T
  constexpr int KCH = 64 * CR;               // chunks in a K tile
  constexpr int VCH = HD * 8;                // chunks in a V^T tile
  constexpr int NBUF = 2;                    // tile buffers per key group (a third one was measured: no gain)
  constexpr int GCH = NBUF * (KCH + VCH);    // chunks per key group
  constexpr int CK = KCH / (QG * 64), CV = VCH / (QG * 64);   // load instructions per wavefront and tile
  constexpr int QB = QG * 32;                // queries per block
  extern __shared__ uint4 smem[];            // per key group: NBUF K tiles, NBUF V^T tiles

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), qt = wave % QG, kg = wave / QG;
  const int lr = lane & 31, lg = lane >> 5;
  // Blocks are dealt round-robin over the 8 XCDs, each with its own L2: give every XCD a contiguous run
  // of (head, query block) work ids so that the blocks streaming one head's K/V share an L2.  The first
  // n_full blocks (a multiple of 8) each own a whole work id; the n_tail work ids after them are cut into
  // `parts` key ranges each, one block per range, again padded to a multiple of 8 blocks that have nothing
  // to do.
  const int NKT = (int)((L + 63) / 64);
  int wid, t0 = 0, t1 = NKT, slot = -1;
  if ((int)blockIdx.x < n_full) {
    wid = (int)(blockIdx.x & 7) * (n_full >> 3) + (int)(blockIdx.x >> 3);
  } else {
    const int local = (int)blockIdx.x - n_full, tail_grid = (int)gridDim.x - n_full;
    const int pid = (local & 7) * (tail_grid >> 3) + (local >> 3);
    if (pid >= n_tail * parts) return;
    wid = n_full + pid / parts;
    if (parts > 1) {
      const int part = pid % parts;
      t0 = (int)((int64_t)part * NKT / parts);
      t1 = (int)((int64_t)(part + 1) * NKT / parts);
      slot = pid;
    }
  }
  const int head = wid / qblocks;
  const int64_t q0 = (int64_t)(wid % qblocks) * QB + qt * 32;
  uint4* const kbuf = smem + kg * GCH;
  uint4* const vbuf = kbuf + NBUF * KCH;

  // this wavefront's key tiles: of two key groups the first has one more if they are odd
  const int n0 = KG == 2 ? (t1 - t0 + 1) / 2 : t1 - t0;          // the trip count for everyone
  const int cnt = kg ? t1 - t0 - n0 : n0;
  t0 += kg ? n0 : 0;

  const bf16_t* kh = k + (int64_t)head * k_head_stride + (k_row0 + (int64_t)t0 * 64) * HD;
  const bf16_t* vh = vt + (int64_t)head * HD * vt_row_stride + k_row0 + (int64_t)t0 * 64;

  // HBM -> LDS directly (no staging registers).  One wavefront instruction fills 64 consecutive
  // 16-byte LDS slots, slot = base + lane; each lane fetches the chunk that belongs in its slot:
  // K slot p holds chunk (p % CR) ^ kswz(row) of key swap23(row), row = p / CR;
  // V^T slot p holds chunk (p % 8) ^ ((row >> 1) & 7) of channel row = p / 8.
  int koff[CK], voff[CV];
#pragma unroll
  for (int i = 0; i < CK; ++i) {
    const int p = qt * (KCH / QG) + i * 64 + lane, row = p / CR, ch = (p % CR) ^ kswz<CR>(row);
    koff[i] = swap23(row) * HD + ch * 8;
  }
#pragma unroll
  for (int i = 0; i < CV; ++i) {
    const int p = qt * (VCH / QG) + i * 64 + lane, row = p >> 3, ch = (p & 7) ^ ((row >> 1) & 7);
    voff[i] = row * (int)vt_row_stride + ch * 8;
  }
  // load instruction i of this wavefront's share of a tile: the K part first (i < CK), then the V^T part
  auto load_part = [&](int tile, int bufi, int i) __attribute__((always_inline)) {
    if (i < CK)
      __builtin_amdgcn_global_load_lds((glb_void_t*)(kh + (int64_t)tile * 64 * HD + koff[i]),
                                       (lds_void_t*)(kbuf + bufi * KCH + qt * (KCH / QG) + i * 64), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds((glb_void_t*)(vh + (int64_t)tile * 64 + voff[i - CK]),
                                       (lds_void_t*)(vbuf + bufi * VCH + qt * (VCH / QG) + (i - CK) * 64), 16, 0, 0);
  };
  auto load_tile = [&](int tile, int bufi) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < CK + CV; ++i) load_part(tile, bufi, i);
  };

  // The queries' row sums, the queries and the fast pass's first two tiles: one trip to memory.  Which goes first decides how the
  // wavefronts of a SIMD stand to each other from then on, and that some per cent of the whole: eight wavefronts on the same tiles
  // want the tiles first (in a stage, queries first / tiles first in us: of 128 3000 x 2000 x 14 60.2 / 58.2, 6240 x 6240 x 12 235 / 225; of 64
  // 3648 x 3648 x 38 159 / 154), two key groups the queries (1560 x 2500 x 12 of 128 46.1 / 47.0), four wavefronts either.
  constexpr bool TILES_FIRST = QG == 8;
  bf16x8 qf[KS];
  QuerySums qs;
  auto request_tiles = [&]() __attribute__((always_inline)) {
    if (cnt > 0) load_tile(cnt - 1, 0);
    if (cnt > 1) load_tile(cnt - 2, 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (TILES_FIRST) request_tiles();
  request_queries<KS, HD>(q + (int64_t)head * q_head_stride, q0, lr, lg, S, qn, qs, qf);
  if constexpr (!TILES_FIRST) request_tiles();
  if (qn.ssq) scale_queries(qf, qs.factor<32>(qn, lg));

  f32x16 oacc[DT], negm;
  float mrun, lsum;

  // Safe pass over this wavefront's key tiles: classical online softmax, reference raised per 32-key half tile, O^T rescaled.
  // Scores of -inf weigh 0 and set no reference: until a query has another (fresh) its reference is 0, and -inf afterwards.
  auto pass_safe = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < DT; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[a][r] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[r] = 0.f;
    mrun = 0.f; lsum = 0.f;
    bool fresh = true;

    if (cnt > 0) load_tile(0, 0);
    tile_barrier();
    for (int kt = 0; kt < n0; ++kt) {
      if (KG == 2 && kt >= cnt) { tile_barrier(); continue; }    // this key group is a tile shorter: it only keeps step
      // next tile into the other buffer (read last before the previous barrier); the tile past the
      // end is the last one again and never used
      load_tile(kt + NBUF - 1 < cnt ? kt + NBUF - 1 : cnt - 1, (kt + NBUF - 1) % NBUF);
      const uint4* kb = kbuf + (kt % NBUF) * KCH;
      const uint4* vb = vbuf + (kt % NBUF) * VCH;
      const int kvalid = (int)(L - (int64_t)(t0 + kt) * 64);     // < 64 only in the ragged last tile
#pragma unroll
      for (int a = 0; a < 2; ++a) {                                  // two 32-key halves of the tile
        // S^T - m : 32 keys x 32 queries, accumulation started from -m
        f32x16 sacc;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const int row = a * 32 + lr, ch = ks * 2 + lg;
          const bf16x8 kf = __builtin_bit_cast(bf16x8, kb[row * CR + (ch ^ kswz<CR>(row))]);
          sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], ks == 0 ? negm : sacc, 0, 0, 0);
        }
        // register r, lane group lg, is tile row a*32 + (r/4)*8 + lg*4 + (r%4), which holds key
        // swap23(row); keys at or beyond L get -inf
        if (kvalid < 64) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (swap23(a * 32 + (r >> 2) * 8 + lg * 4 + (r & 3)) >= kvalid) sacc[r] = -INFINITY;
        }
        float mx = sacc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sacc[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));                    // maximum of this half relative to m
        const bool none = mx == -INFINITY;
        const float up = none ? 0.f : fresh ? mx : fmaxf(mx, 0.f);
        const float alpha = fresh ? 0.f : __builtin_amdgcn_exp2f(-up);
        mrun += up;
        lsum *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) { sacc[r] -= up; negm[r] = -mrun; }
        fresh = fresh && none;
        // P = 2^(s - m), packed to bf16 as the B operand of O^T += V^T P^T; row sums from the rounded values
        uint4 pf[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          uint32_t w[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            w[j] = cvt_pk_bf16(__builtin_amdgcn_exp2f(sacc[u * 8 + 2 * j]), __builtin_amdgcn_exp2f(sacc[u * 8 + 2 * j + 1]));
            lsum = add_pk_bf16(w[j], lsum);
          }
          pf[u] = make_uint4(w[0], w[1], w[2], w[3]);
        }
        // O^T += V^T * P^T : k-step u covers keys [a*32 + 16u, +16), lane group lg the lower/upper 8
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            const int row = dt * 32 + lr, ch = (a * 2 + u) * 2 + lg;
            const bf16x8 vf = __builtin_bit_cast(bf16x8, vb[row * 8 + (ch ^ ((row >> 1) & 7))]);
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pf[u]), oacc[dt], 0, 0, 0);
          }
        }
      }
      tile_barrier();       // the next tile has landed and every wavefront is done with this one
    }
    if (fresh) mrun = -INFINITY;
  };

  // Fast pass (fixed reference).  Per tile a wavefront issues NMF MFMAs in the order S^T of the first 32-key
  // half, S^T of the second half, O^T += V^T P^T of the first half, then of the second; the exponentials of
  // the first half are issued between the MFMAs of the second half's S^T and those of the second half
  // between the first half's V^T P^T MFMAs, so the vector unit works while the matrix pipe runs.  Every MFMA
  // takes one operand fragment from LDS; fragment i + PD is read right behind MFMA i, through inline
  // assembly with explicit waits (LDS returns reads in order), so an MFMA never waits for a read issued
  // just before it.  The tile's barrier sits PD MFMAs before the tile's end, once all its fragments are in
  // registers: behind it the loads of the tile after next and the first PD fragment reads of the next tile
  // go out between the remaining MFMAs.
  constexpr int NMF = 2 * (KS + 2 * DT), PD = 4, PPM = 8 / KS;      // MFMAs per tile, read-ahead, exp pairs per MFMA
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  // This lane's row of a K tile (row lr of a 32-key half) and of a V^T tile (row lr of a 32-channel group) in
  // buffer 0, as LDS byte addresses; chunk c of the row sits at byte (c * 16) ^ swizzle, and c = ks*2 + lg or
  // (a*2+u)*2 + lg has lg as its lowest bit, so the lane-dependent part of the XOR is one constant per tile kind.
  const uint32_t krow = lds0 + (uint32_t)(kg * GCH + lr * CR) * 16, kx = (uint32_t)(lg ^ kswz<CR>(lr)) * 16;
  const uint32_t vrow = lds0 + (uint32_t)(kg * GCH + NBUF * KCH + lr * 8) * 16, vx = (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;
  // operand fragment of MFMA i of a tile whose K / V^T buffers start kbo / vbo bytes behind buffer 0
  auto frag_read = [&](auto i_, uint32_t kbo, uint32_t vbo) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value;
    if constexpr (i < 2 * KS) {
      return lds_read16<(i / KS) * 32 * CR * 16>((krow + kbo) + (kx ^ (uint32_t)((i % KS) * 32)));
    } else {
      constexpr int j = i - 2 * KS, a = j / (2 * DT), u = (j % (2 * DT)) / DT, dt = j % DT;
      return lds_read16<dt * 32 * 8 * 16>((vrow + vbo) + (vx ^ (uint32_t)((a * 2 + u) * 32)));
    }
  };
  auto pass_fast = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < DT; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[a][r] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[r] = 0.f;
    mrun = 0.f; lsum = 0.f;
    // Step j of this pass works on tile cnt - 1 - j of the range (the sums do not care about the order), in
    // buffer j % NBUF (the first two are on their way): the last tile of the range, the only one that can be ragged, comes first and is done
    // here in plain order with its keys at or beyond L masked; the pinned loop below then sees whole tiles only.
    tile_barrier();
    if (cnt > 0) {
      const int kvalid = (int)(L - (int64_t)(t0 + cnt - 1) * 64);   // >= 1; < 64 only in a ragged tile
      // reference = maximum over the tile's first 32 keys (the valid ones of them).  Register r of lane group
      // lg is tile row a*32 + (r/4)*8 + lg*4 + r%4, which holds key swap23(row).
      f32x16 sv;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int row = lr, ch = ks * 2 + lg;
        const bf16x8 kf = __builtin_bit_cast(bf16x8, kbuf[row * CR + (ch ^ kswz<CR>(row))]);
        sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], ks == 0 ? negm : sv, 0, 0, 0);
      }
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (swap23((r >> 2) * 8 + lg * 4 + (r & 3)) < kvalid) mx = fmaxf(mx, sv[r]);
      mrun = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll
      for (int r = 0; r < 16; ++r) negm[r] = -mrun;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        if (a == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) sv[r] -= mrun;
        } else {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const int row = 32 + lr, ch = ks * 2 + lg;
            const bf16x8 kf = __builtin_bit_cast(bf16x8, kbuf[row * CR + (ch ^ kswz<CR>(row))]);
            sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], ks == 0 ? negm : sv, 0, 0, 0);
          }
        }
        if (kvalid < 64) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (swap23(a * 32 + (r >> 2) * 8 + lg * 4 + (r & 3)) >= kvalid) sv[r] = -INFINITY;
        }
        uint4 pf[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          uint32_t w[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            w[j] = cvt_pk_bf16(__builtin_amdgcn_exp2f(sv[u * 8 + 2 * j]), __builtin_amdgcn_exp2f(sv[u * 8 + 2 * j + 1]));
            lsum = add_pk_bf16(w[j], lsum);
          }
          pf[u] = make_uint4(w[0], w[1], w[2], w[3]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            const int row = dt * 32 + lr, ch = (a * 2 + u) * 2 + lg;
            const bf16x8 vf = __builtin_bit_cast(bf16x8, vbuf[row * 8 + (ch ^ ((row >> 1) & 7))]);
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pf[u]), oacc[dt], 0, 0, 0);
          }
      }
    }
    tile_barrier();                 // every wavefront is done with buffer 0
    if (cnt > 2) load_tile(cnt - 3, 0);
    bf16x8 fr[PD];
    f32x16 sacc[2];
    uint32_t pw[2][8];              // P of the two halves: packed bf16 pairs, four per MFMA operand
    static_for<PD>([&](auto i_) __attribute__((always_inline)) {
      fr[decltype(i_)::value] = frag_read(i_, (uint32_t)(1 % NBUF) * KCH * 16, (uint32_t)(1 % NBUF) * VCH * 16);
    });
    // exponentials of scores 2p, 2p+1 of half a, packed; row sums from the rounded values
    auto e_piece = [&](int a, int pidx) __attribute__((always_inline)) {
      pw[a][pidx] = cvt_pk_bf16(__builtin_amdgcn_exp2f(sacc[a][2 * pidx]), __builtin_amdgcn_exp2f(sacc[a][2 * pidx + 1]));
      lsum = add_pk_bf16(pw[a][pidx], lsum);
    };
    for (int j = 1; j < n0; ++j) {
      // a key group that is a tile shorter only keeps step.  With one group that is never so, but heads of 64 run 2 % faster with the
      // branch, by which the compiler lays out the loop, and heads of 128 2 % slower.
      if ((KG == 2 || (HD == 64 && QG == 8)) && j >= cnt) { tile_barrier(); continue; }
      const uint32_t kbo = (uint32_t)(j % NBUF) * KCH * 16, vbo = (uint32_t)(j % NBUF) * VCH * 16;
      const uint32_t kbn = (uint32_t)((j + 1) % NBUF) * KCH * 16, vbn = (uint32_t)((j + 1) % NBUF) * VCH * 16;
      static_for<NMF>([&](auto i_) __attribute__((always_inline)) {
        constexpr int i = decltype(i_)::value;
        if constexpr (i < NMF - PD) lds_wait<PD - 1>();               // fragment i has landed
        __builtin_amdgcn_sched_barrier(0);                            // the MFMA stays behind the wait
        if constexpr (i < KS) {
          sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % PD], qf[i], i == 0 ? negm : sacc[0], 0, 0, 0);
        } else if constexpr (i < 2 * KS) {
          sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % PD], qf[i - KS], i == KS ? negm : sacc[1], 0, 0, 0);
#pragma unroll
          for (int e = 0; e < PPM; ++e) e_piece(0, (i - KS) * PPM + e);
        } else {
          constexpr int m = i - 2 * KS, a = m / (2 * DT), u = (m % (2 * DT)) / DT, dt = m % DT;
          const uint4 pf = make_uint4(pw[a][u * 4], pw[a][u * 4 + 1], pw[a][u * 4 + 2], pw[a][u * 4 + 3]);
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % PD], __builtin_bit_cast(bf16x8, pf), oacc[dt], 0, 0, 0);
          if constexpr (a == 0) {
#pragma unroll
            for (int e = 0; e < PPM; ++e) e_piece(1, m * PPM + e);
          }
        }
        // the two dependent S^T chains go first in the SIMD's issue arbitration (measured: 2 % over no hint)
        if constexpr (i == 0) __builtin_amdgcn_s_setprio(1);
        if constexpr (i == 2 * KS - 1) __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);      // the read that reuses the MFMA's operand register stays behind it
        if constexpr (i + PD < NMF) fr[i % PD] = frag_read(std::integral_constant<int, i + PD>{}, kbo, vbo);
        if constexpr (i == NMF - PD - 1) {
          lds_wait<0>();          // every fragment of this tile is in registers
          tile_barrier();         // the next tile has landed and every wavefront is done reading this one
        }
        if constexpr (i >= NMF - PD) {
          if (j + 2 < cnt) {
#pragma unroll
            for (int q = 0; q < CK + CV; ++q)
              if (q * PD / (CK + CV) == i - (NMF - PD)) load_part(cnt - 3 - j, j % NBUF, q);
          }
          fr[i % PD] = frag_read(std::integral_constant<int, i + PD - NMF>{}, kbn, vbn);
        }
        __builtin_amdgcn_sched_barrier(0);                            // keeps this order
      });
    }
    lds_wait<0>();
  };

  pass_fast();
  float ltot = lsum + __shfl_xor(lsum, 32, 64);
  if (__syncthreads_or(!(ltot <= 0x1p100f))) {          // overflow somewhere in the block: redo it safely
    pass_safe();
    ltot = lsum + __shfl_xor(lsum, 32, 64);
  }
  if constexpr (KG == 2) {
    // the two key groups meet in LDS: group 1 publishes m, l, O^T, and group 0 goes on with both
    float* const xch = (float*)smem + (size_t)qt * (DT * 16 + 2) * 64 + lane;    // [qt][DT * 16 + 2][64 lanes]
    if (kg == 1) {
      xch[0] = mrun; xch[64] = ltot;
#pragma unroll
      for (int a = 0; a < DT; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) xch[(2 + a * 16 + r) * 64] = oacc[a][r];
    }
    __syncthreads();
    if (kg == 1) return;
    const float m1 = xch[0], l1 = xch[64], m = fmaxf(mrun, m1);
    const float ref = m == -INFINITY ? 0.f : m;          // a range of nothing but -inf: l and O stay 0
    const float a0 = __builtin_amdgcn_exp2f(mrun - ref), a1 = __builtin_amdgcn_exp2f(m1 - ref);
    mrun = m;
    ltot = ltot * a0 + l1 * a1;
#pragma unroll
    for (int a = 0; a < DT; ++a)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[a][r] = oacc[a][r] * a0 + xch[(2 + a * 16 + r) * 64] * a1;
  }
  if (slot >= 0) {
    // one key range of a split work id: publish m, l and the unnormalised O^T for the merge kernel.
    // Slot layout (floats): m[QB], l[QB], then O as [HD/4][QB queries][4 channels].
    float* ps = partial + (size_t)slot * (2 * QB + QB * HD);
    const int ql = qt * 32 + lr;
    if (lg == 0) { ps[ql] = mrun; ps[QB + ql] = ltot; }
#pragma unroll
    for (int a = 0; a < DT; ++a)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float4 v = make_float4(oacc[a][g4 * 4 + 0], oacc[a][g4 * 4 + 1], oacc[a][g4 * 4 + 2], oacc[a][g4 * 4 + 3]);
        *(float4*)(ps + 2 * QB + ((size_t)(a * 8 + g4 * 2 + lg) * QB + ql) * 4) = v;
      }
  } else {
    // O[q][head*HD + c] = O^T[c][q]: a lane holds 4 consecutive channels per register quad.  The 32 x HD
    // tile of this wavefront goes through LDS (the tile buffers are free; a wavefront only touches its own
    // rows, and LDS serves a wavefront's accesses in order) so that global memory sees whole rows, 16
    // bytes per lane.  8-byte units are XOR-swizzled with the row so that the column-wise writes spread
    // over the banks.
    const float inv = 1.f / ltot;
    constexpr int UPR = HD / 4, CPR = HD / 8, RPI = 64 / CPR;      // units, 16-byte chunks per row; rows per read
    constexpr int STG0 = KG == 2 ? QG * (DT * 16 + 2) * 64 / 4 : 0;    // behind the exchange area
    uint2* stg = (uint2*)(smem + STG0) + qt * 32 * UPR;
#pragma unroll
    for (int a = 0; a < DT; ++a)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        uint2 pk;
        pk.x = cvt_pk_bf16(oacc[a][g4 * 4 + 0] * inv, oacc[a][g4 * 4 + 1] * inv);
        pk.y = cvt_pk_bf16(oacc[a][g4 * 4 + 2] * inv, oacc[a][g4 * 4 + 3] * inv);
        stg[lr * UPR + ((a * 8 + g4 * 2 + lg) ^ (lr & (UPR - 1)))] = pk;
      }
    const uint4* stg16 = (const uint4*)stg;
#pragma unroll
    for (int it = 0; it < 32 / RPI; ++it) {
      const int row = it * RPI + lane / CPR, p = lane % CPR;
      uint4 dv = stg16[row * CPR + p];
      // units 2p and 2p+1 of the swizzled row are the halves of chunk p ^ (swizzle >> 1), exchanged for odd rows
      if (row & 1) dv = make_uint4(dv.z, dv.w, dv.x, dv.y);
      const int c = p ^ ((row & (UPR - 1)) >> 1);
      if (q0 + row < S) *(uint4*)(out + (q0 + row) * ldo + (int64_t)head * HD + c * 8) = dv;
    }
  }
}

// Eight wavefronts of 32 queries (two MFMA columns of 16), v_mfma_f32_16x16x32_bf16, key tiles of 64.  KG = 1: all share every
// tile, a block has 256 queries and its halves are the wavefronts 0-3 and 4-7.  KG = 2: the halves have the same 128 queries
// and one part of the keys each, with tiles of their own; they meet in LDS at the end, which halves the length of a block.
// The two wavefronts of a SIMD (one of each half) take turns, with a barrier at every change: one multiplies, the scores of
// tile j + 1 and the weighted sum of tile j back to back, and reads tile j's V^T fragments into the registers that the keys
// leave; the other turns its scores of tile j + 1 into weights, reads tile j + 2's keys and requests tiles to come.  A turn of
// products is 64 MFMAs of 16 cycles at head_dim 128, one of exponentials about 0.7 of that, so the matrix pipes see one
// wavefront or the other all the time; the exponentials have no MFMA to wait for and nothing is interleaved by hand.
// What bounds it: matrix pipes under the power limit.  Against a pinned order in which each wavefront mixed its own
// exponentials between its MFMAs (32x32x16; us): 14400 x 21600 x 40 of 128 4978 -> 4487 (1.42 PFLOP/s), 6240 x 9360 x 12 305 -> 278,
// 7800 x 7800 x 12 314 -> 287, 18720 x 24960 x 12 2250 -> 2026; two key groups 1560 x 3120 x 12 43.6 -> 40.8, 3000 x 4000 x 8 55.9 -> 50.6.  Back to back and alone, that is: in
// a stage and with few keys it is the other way round (attn_bf16_turns).  <128, 2> spills 8 registers outside its loop.
// Tried: loads behind the exponentials (2 % slower), without s_setprio (0.4 %).
template <int HD, int KG>
__global__ __launch_bounds__(512) void k_attn_turns(const bf16_t* __restrict__ q, int64_t q_head_stride,
                                                    const bf16_t* __restrict__ k, int64_t k_head_stride,
                                                    int64_t k_row0, const bf16_t* __restrict__ vt,
                                                    int64_t vt_row_stride, int64_t S, int64_t L,
                                                    bf16_t* __restrict__ out, int64_t ldo, int qblocks,
                                                    int n_full, int n_tail, int parts,
                                                    float* __restrict__ partial, AttnQNorm qn) {
  constexpr int CR = HD / 8;                 // 16-byte chunks per K row
  constexpr int KS = HD / 32, DT = HD / 16;  // MFMA k-steps over the head dim, 16-channel tiles of O^T
  constexpr int KCH = 64 * CR, VCH = HD * 8; // chunks in a K tile and in a V^T tile of 64 keys
  constexpr int QG = 8 / KG, QB = QG * 32;   // wavefronts that share a tile; queries per block
  constexpr int NST = KG == 1 ? 4 : 2;       // LDS stages of either, per key group
  constexpr int CK = KCH / (QG * 64), CV = VCH / (QG * 64);   // load instructions per wavefront and tile
  extern __shared__ uint4 smem[];            // per key group: NST K tiles, NST V^T tiles
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), qt = wave % QG, kg = wave / QG;
  // Work ids as in k_attn_bf16.
  const int NKT = (int)((L + 63) / 64);
  int wid, t0 = 0, t1 = NKT, slot = -1;
  if ((int)blockIdx.x < n_full) {
    wid = (int)(blockIdx.x & 7) * (n_full >> 3) + (int)(blockIdx.x >> 3);
  } else {
    const int local = (int)blockIdx.x - n_full, tail_grid = (int)gridDim.x - n_full;
    const int pid = (local & 7) * (tail_grid >> 3) + (local >> 3);
    if (pid >= n_tail * parts) return;
    wid = n_full + pid / parts;
    if (parts > 1) {
      const int part = pid % parts;
      t0 = (int)((int64_t)part * NKT / parts);
      t1 = (int)((int64_t)(part + 1) * NKT / parts);
      slot = pid;
    }
  }
  // this wavefront's tiles: of two key groups the first has one more if they are odd
  const int n0 = KG == 2 ? (t1 - t0 + 1) / 2 : t1 - t0;          // the trip count for everyone
  const int cnt = kg ? t1 - t0 - n0 : n0;                        // >= 1
  t0 += kg ? n0 : 0;
  const int head = wid / qblocks;
  const int64_t q0 = (int64_t)(wid % qblocks) * QB + qt * 32;
  uint4* const kst = smem + kg * NST * (KCH + VCH);
  uint4* const vst = kst + NST * KCH;
  const bf16_t* const kh = k + (int64_t)head * k_head_stride + (k_row0 + (int64_t)t0 * 64) * HD;
  const bf16_t* const vh = vt + (int64_t)head * HD * vt_row_stride + k_row0 + (int64_t)t0 * 64;

  // K slot p of a tile holds chunk (p % CR) ^ kswz(row) of key keyat(row), row = p / CR; V^T slot p holds chunk
  // (p % 8) ^ ((row >> 1) & 7) of channel row = p / 8.  Tile row u * 16 + g * 4 + r of a 32-key half holds key g * 8 + u * 4 + r, so
  // that the accumulators a lane packs into one operand are eight consecutive keys.
  auto keyat = [](int row) __attribute__((always_inline)) { return (row & 32) | ((row >> 2) & 3) * 8 | ((row >> 4) & 1) * 4 | (row & 3); };
  // A wavefront's load instructions of a tile are QG * 64 slots apart: 16 keys (in rows of 8 or 16 chunks, tile rows 16 or 32
  // apart) or 32 channels and more, so their swizzle is the same and what differs is uniform.
  constexpr int KR = QG * 64 / CR, VR = QG * 8;
  static_assert(KR % 16 == 0 && VR % 16 == 0, "one swizzle");
  const int p0 = qt * 64 + lane;
  const uint32_t koff = (uint32_t)(keyat(p0 / CR) * HD + ((p0 % CR) ^ kswz<CR>(p0 / CR)) * 8) * 2;
  const uint32_t voff = (uint32_t)((p0 >> 3) * vt_row_stride + ((p0 & 7) ^ ((p0 >> 4) & 7)) * 8) * 2;
  // tile j of the walk is tile cnt - 1 - j of the range: the last tile of the range, the only one that can be ragged, comes
  // first; past the end the range's first tile is loaded again and never read
  auto tile_of = [&](int j) __attribute__((always_inline)) { return j < cnt ? cnt - 1 - j : 0; };
  auto load_k = [&](int j) __attribute__((always_inline)) {
    const bf16_t* const base = kh + (int64_t)tile_of(j) * 64 * HD;
#pragma unroll
    for (int i = 0; i < CK; ++i) load_lds16(base, 0x7fffffff, koff, keyat(i * KR) * HD * 2, kst + (j % NST) * KCH + (i * QG + qt) * 64);
  };
  auto load_v = [&](int j) __attribute__((always_inline)) {
    const bf16_t* const base = vh + (int64_t)tile_of(j) * 64;
#pragma unroll
    for (int i = 0; i < CV; ++i) load_lds16(base, 0xffffffff, voff, (int)((uint32_t)(i * VR * 2) * (uint32_t)vt_row_stride), vst + (j % NST) * VCH + (i * QG + qt) * 64);
  };
  // one trip to memory: the queries' row sums, the queries, the tiles in the order in which they are needed
  QuerySums qs[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) qs[t].request(qn, q0 + t * 16 + lr, S, lg & 1);
  // the fragments of this wavefront's 32 queries: B operand, column = query lr of a 16-query tile, 8 head-dim values per lane
  bf16x8 qf[2][KS];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const bf16_t* const qh = q + (int64_t)head * q_head_stride + (q0 + t * 16 + lr) * HD + lg * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[t][ks] = __builtin_bit_cast(bf16x8, *(const uint4*)(qh + ks * 32));
  }
  __builtin_amdgcn_sched_barrier(0);
  load_k(0); load_k(1);
  load_v(0);
  if constexpr (KG == 1) { load_k(2); load_v(1); load_k(3); } else load_v(1);
  __builtin_amdgcn_sched_barrier(0);
  if (qn.ssq) {
#pragma unroll
    for (int t = 0; t < 2; ++t) scale_queries(qf[t], qs[t].factor<16>(qn, lg & 1));
  }
  __builtin_amdgcn_sched_barrier(0);

  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  const uint32_t krow = lds0 + (uint32_t)(kg * NST * (KCH + VCH) + lr * CR) * 16, kx = (uint32_t)(lg ^ kswz<CR>(lr)) * 16;
  const uint32_t vrow = lds0 + (uint32_t)(kg * NST * (KCH + VCH) + NST * KCH + lr * 8) * 16, vx = (uint32_t)(lg ^ ((lr >> 1) & 7)) * 16;
  bf16x8 kf[4][KS], vf[2][DT];
  f32x4 o[DT][2], sc[4][2], negm[2];
  uint4 pf[2][2];                            // P of a tile: [32-key half][query tile], packed
  float lsum[2];
  // 16-byte fragments of key tile j: keys kt * 16 .., head-dim values ks * 32 ..
  auto read_k = [&](int j) __attribute__((always_inline)) {
    const uint32_t b = krow + (uint32_t)(j % NST) * KCH * 16;
    static_for<KS>([&](auto k_) __attribute__((always_inline)) {
      constexpr int ks = decltype(k_)::value;
      static_for<4>([&](auto t_) __attribute__((always_inline)) {
        constexpr int t = decltype(t_)::value;
        kf[t][ks] = lds_read16<t * 16 * CR * 16>(b + (kx ^ (uint32_t)(ks * 64)));
      });
    });
  };
  // four of the fragments of V^T tile j, in the order in which they are used
  auto read_v4 = [&](int j, auto g_) __attribute__((always_inline)) {
    constexpr int g = decltype(g_)::value;
    const uint32_t b = vrow + (uint32_t)(j % NST) * VCH * 16;
    static_for<4>([&](auto i_) __attribute__((always_inline)) {
      constexpr int f = g * 4 + decltype(i_)::value, s = f / DT, d = f % DT;
      vf[s][d] = lds_read16<d * 16 * 8 * 16>(b + (vx ^ (uint32_t)(s * 64)));
    });
  };
  // this lane's key of accumulator register r of 16-key tile t
  auto key_of = [&](int t, int r) __attribute__((always_inline)) { return (t >> 1) * 32 + lg * 8 + (t & 1) * 4 + r; };
  // P = 2^(s - m) of the tile in sc, rounded to bf16 and packed; row sums from the rounded values
  auto weigh = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4& v = sc[2 * s + (i >> 1)][t];
          w[i] = cvt_pk_bf16(__builtin_amdgcn_exp2f(v[2 * (i & 1)]), __builtin_amdgcn_exp2f(v[2 * (i & 1) + 1]));
          lsum[t] = add_pk_bf16(w[i], lsum[t]);
        }
        pf[s][t] = make_uint4(w[0], w[1], w[2], w[3]);
      }
  };
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int t = 0; t < 2; ++t) o[d][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    lsum[0] = lsum[1] = 0.f;
  };
  auto scores = [&](bool from_zero) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          sc[kt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kt][ks], qf[t][ks], ks == 0 ? (from_zero ? f32x4{0.f, 0.f, 0.f, 0.f} : negm[t]) : sc[kt][t], 0, 0, 0);
  };
  // maximum of sc[kt][t] over kt0 <= kt < kt1 and the four lanes of a query
  auto maximum = [&](int t, int kt1) __attribute__((always_inline)) {
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
      if (kt < kt1)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sc[kt][t][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    return fmaxf(mx, __shfl_xor(mx, 32, 64));
  };
  auto mask = [&](int kvalid) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (key_of(kt, r) >= kvalid) { sc[kt][0][r] = -INFINITY; sc[kt][1][r] = -INFINITY; }
  };

  // Tile 0, in plain order: its scores, the reference of every query (its maximum over the tile's first 32 keys, the valid ones
  // of them), its weights; and tile 1's keys
  clear();
  vm_wait<KG == 1 ? 2 * (CK + CV) : 2 * CV>();   // K tiles 0 and 1
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  read_k(0);
  lds_wait<0>();
  __builtin_amdgcn_sched_barrier(0);
  scores(true);
  const int kvalid = (int)(L - (int64_t)(t0 + cnt - 1) * 64);    // of tile 0: >= 1, < 64 only if it is ragged
  if (kvalid < 64) mask(kvalid);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const float m = maximum(t, 2);
#pragma unroll
    for (int r = 0; r < 4; ++r) negm[t][r] = -m;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) sc[kt][t] += negm[t];
  }
  weigh();
  __builtin_amdgcn_sched_barrier(0);
  read_k(1);
  lds_wait<0>();
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();                           // K stage 0 is free
  if constexpr (KG == 1) { load_v(2); load_k(4); } else load_k(2);
  vm_wait<KG == 1 ? CK + CV : CK>();         // V tiles 0 and 1, and K tiles 2 and 3 of four stages
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  if (wave >= 4) __builtin_amdgcn_s_barrier();   // the second half starts half a turn later
  __builtin_amdgcn_sched_barrier(0);
  for (int j = 0; j < n0 - 1; ++j) {
    if (KG == 2 && j >= cnt - 1) {           // this key group is a tile shorter: it only keeps step
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_s_barrier();
      continue;
    }
    // scores of tile j + 1 and the weighted sum of tile j, whose V^T fragments take the place of the used keys
    __builtin_amdgcn_s_setprio(1);
    static_for<KS>([&](auto k_) __attribute__((always_inline)) {
      constexpr int ks = decltype(k_)::value;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          sc[kt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kt][ks], qf[t][ks], ks == 0 ? negm[t] : sc[kt][t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (ks > 0) read_v4(j, std::integral_constant<int, ks - 1>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<KS>([&](auto g_) __attribute__((always_inline)) {
      constexpr int g = decltype(g_)::value;
      lds_wait<4 * (g == 0 ? KS - 2 : KS - 1 - g)>();
      __builtin_amdgcn_sched_barrier(0);
      static_for<4>([&](auto i_) __attribute__((always_inline)) {
        constexpr int f = g * 4 + decltype(i_)::value, s = f / DT, d = f % DT;
#pragma unroll
        for (int t = 0; t < 2; ++t) o[d][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[s][d], __builtin_bit_cast(bf16x8, pf[s][t]), o[d][t], 0, 0, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (g == 0) read_v4(j, std::integral_constant<int, KS - 1>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (KG == 2) vm_wait<0>();     // K tile j + 2, requested two turns ago
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // the other half multiplies: tile j + 2's keys, tiles to come, weights of tile j + 1
    read_k(j + 2);
    __builtin_amdgcn_sched_barrier(0);
    // into stages that this group's wavefronts (one group: both halves) have read
    if constexpr (KG == 1) { load_v(j + 3); load_k(j + 5); } else { load_v(j + 2); load_k(j + 3); }
    __builtin_amdgcn_sched_barrier(0);
    weigh();
    if constexpr (KG == 1) vm_wait<CK + CV>();   // what was requested before this turn: V tile j + 2, K tile j + 4
    lds_wait<0>();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }
  // the last tile's weighted sum
  static_for<KS>([&](auto g_) __attribute__((always_inline)) { read_v4(cnt - 1, g_); });
  lds_wait<0>();
  __builtin_amdgcn_sched_barrier(0);
  static_for<2>([&](auto s_) __attribute__((always_inline)) {
    constexpr int s = decltype(s_)::value;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int t = 0; t < 2; ++t) o[d][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[s][d], __builtin_bit_cast(bf16x8, pf[s][t]), o[d][t], 0, 0, 0);
  });
  if (wave < 4) __builtin_amdgcn_s_barrier();    // the halves meet again
  __builtin_amdgcn_sched_barrier(0);
  tile_barrier();                            // nothing is in flight any more

  auto total = [&](float v) __attribute__((always_inline)) { v += __shfl_xor(v, 16, 64); return v + __shfl_xor(v, 32, 64); };
  float ltot[2] = {total(lsum[0]), total(lsum[1])};
  if (__syncthreads_or(!(ltot[0] <= 0x1p100f) || !(ltot[1] <= 0x1p100f))) {
    // overflow somewhere in the block: the classical online softmax, tile by tile
    clear();
#pragma unroll
    for (int t = 0; t < 2; ++t) negm[t][0] = INFINITY;
    for (int j = 0; j < n0; ++j) {
      __syncthreads();
      load_k(j); load_v(j);
      tile_barrier();
      if (KG == 2 && j >= cnt) continue;
      read_k(j);
      static_for<KS>([&](auto g_) __attribute__((always_inline)) { read_v4(j, g_); });
      lds_wait<0>();
      __builtin_amdgcn_sched_barrier(0);
      scores(true);
      if (j == 0 && kvalid < 64) mask(kvalid);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        // no key above -inf yet: any finite reference leaves zero weights
        const float m = fmaxf(maximum(t, 4), -negm[t][0]), ref = m == -INFINITY ? 0.f : m;
        const float alpha = __builtin_amdgcn_exp2f(-negm[t][0] - ref);
        negm[t][0] = -m;
        lsum[t] *= alpha;
#pragma unroll
        for (int d = 0; d < DT; ++d) o[d][t] *= alpha;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) sc[kt][t] -= ref;
      }
      weigh();
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
          for (int t = 0; t < 2; ++t) o[d][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[s][d], __builtin_bit_cast(bf16x8, pf[s][t]), o[d][t], 0, 0, 0);
    }
    ltot[0] = total(lsum[0]); ltot[1] = total(lsum[1]);
    __syncthreads();
  }

  float mrun[2] = {-negm[0][0], -negm[1][0]};
  float4* const xch = (float4*)smem + (size_t)qt * (2 * DT + 1) * 64 + lane;     // [qt][2 * DT + 1][64 lanes]
  if constexpr (KG == 2) {
    // the two key groups meet in LDS: group 1 publishes m, l, O^T, and group 0 goes on with both
    if (kg == 1) {
      xch[0] = make_float4(mrun[0], mrun[1], ltot[0], ltot[1]);
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int t = 0; t < 2; ++t) xch[(1 + 2 * d + t) * 64] = make_float4(o[d][t][0], o[d][t][1], o[d][t][2], o[d][t][3]);
    }
    __syncthreads();
    if (kg == 1) return;
    const float4 ml = xch[0];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float m1 = t ? ml.y : ml.x, l1 = t ? ml.w : ml.z, m = fmaxf(mrun[t], m1);
      const float ref = m == -INFINITY ? 0.f : m;          // a range of nothing but -inf: l and O stay 0
      const float a0 = __builtin_amdgcn_exp2f(mrun[t] - ref), a1 = __builtin_amdgcn_exp2f(m1 - ref);
      mrun[t] = m;
      ltot[t] = ltot[t] * a0 + l1 * a1;
#pragma unroll
      for (int d = 0; d < DT; ++d) {
        const float4 v = xch[(1 + 2 * d + t) * 64];
        o[d][t] = o[d][t] * a0 + f32x4{v.x, v.y, v.z, v.w} * a1;
      }
    }
  }
  if (slot >= 0) {
    // one key range of a split work id: publish m, l and the unnormalised O^T for the merge kernel.
    // Slot layout (floats): m[QB], l[QB], then O as [HD/4][QB queries][4 channels].
    float* ps = partial + (size_t)slot * (2 * QB + QB * HD);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int ql = qt * 32 + t * 16 + lr;
      if (lg == 0) { ps[ql] = mrun[t]; ps[QB + ql] = ltot[t]; }
#pragma unroll
      for (int d = 0; d < DT; ++d) *(f32x4*)(ps + 2 * QB + ((size_t)(d * 4 + lg) * QB + ql) * 4) = o[d][t];
    }
  } else {
    // O[q][head*HD + c] = O^T[c][q]: a lane holds 4 consecutive channels per accumulator tile.  The 32 x HD tile of this
    // wavefront goes through LDS (a wavefront only touches its own rows, and LDS serves a wavefront's accesses in order) so that
    // global memory sees whole rows, 16 bytes per lane.  8-byte units are XOR-swizzled with the row.
    constexpr int UPR = HD / 4, CPR = HD / 8, RPI = 64 / CPR;      // units, 16-byte chunks per row; rows per read
    constexpr int STG0 = KG == 2 ? QG * (2 * DT + 1) * 64 : 0;     // behind the exchange area
    uint2* stg = (uint2*)(smem + STG0) + qt * 32 * UPR;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float inv = 1.f / ltot[t];
      const int row = t * 16 + lr;
#pragma unroll
      for (int d = 0; d < DT; ++d)
        stg[row * UPR + ((d * 4 + lg) ^ (row & (UPR - 1)))] = make_uint2(cvt_pk_bf16(o[d][t][0] * inv, o[d][t][1] * inv), cvt_pk_bf16(o[d][t][2] * inv, o[d][t][3] * inv));
    }
    const uint4* stg16 = (const uint4*)stg;
#pragma unroll
    for (int it = 0; it < 32 / RPI; ++it) {
      const int row = it * RPI + lane / CPR, p = lane % CPR;
      uint4 dv = stg16[row * CPR + p];
      // units 2p and 2p+1 of the swizzled row are the halves of chunk p ^ (swizzle >> 1), exchanged for odd rows
      if (row & 1) dv = make_uint4(dv.z, dv.w, dv.x, dv.y);
      const int c = p ^ ((row & (UPR - 1)) >> 1);
      if (q0 + row < S) *(uint4*)(out + (q0 + row) * ldo + (int64_t)head * HD + c * 8) = dv;
    }
  }
}

// Few queries against few keys.  A block owns 32 queries of one head and its 8 wavefronts deal the key range out in tiles
// of 32 keys (wavefront w: tiles w, w + 8, ...), each through its own piece of LDS and with its own online softmax; nobody
// waits for anybody until the eight partial results are added up in LDS, in wavefront order.  What bounds it is latency: the
// launch, one trip to memory, two short MFMA chains and the sum; k_attn_bf16 spends 4.5 us on its two groups' tile-by-tile
// barriers, reference pass and merge around the tiles, and 1.5 us for every two tiles of 64 keys.  Measured (us, back to back;
// queries x keys x heads): head_dim 128 216 x 360 x 2 11.9 -> 8.1, 216 x 40 x 2 8.6 -> 5.1, 500 x 700 x 4 15.7 -> 10.4; head_dim 64
// 333 x 1000 x 12 13.2 -> 8.7, 1008 x 77 x 16 6.9 -> 5.8.
template <int HD>
__global__ __launch_bounds__(512, HD == 64 ? 4 : 2) void k_attn_few(const bf16_t* __restrict__ q, int64_t q_head_stride, const bf16_t* __restrict__ k,
                                                 int64_t k_head_stride, int64_t k_row0, const bf16_t* __restrict__ vt,
                                                 int64_t vt_row_stride, int64_t S, int64_t L, bf16_t* __restrict__ out,
                                                 int64_t ldo, int qblocks, int n_work, AttnQNorm qn) {
  constexpr int CR = HD / 8, KS = HD / 16, DT = HD / 32, QB = 32;
  constexpr int KCH = 32 * CR, VCH = HD * 4;             // 16-byte chunks of a K tile (32 keys) and of a V^T tile
  constexpr int OCH = QB * HD / 4;                       // of a partial result: fp32 [QB][HD]
  constexpr int MINE = KCH + VCH > OCH ? KCH + VCH : OCH;
  extern __shared__ uint4 smem[];                        // 8 * MINE chunks
  __shared__ float2 ml[8][QB];                           // reference and row sum of each wavefront's part
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wid = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);   // contiguous per XCD
  if (wid >= n_work) return;
  const int head = wid / qblocks;
  const int64_t q0 = (int64_t)(wid % qblocks) * QB;
  const int NT = (int)((L + 31) / 32), parts = NT < 8 ? NT : 8;
  uint4* const mine = smem + wave * MINE;

  if (wave < parts) {
    const bf16_t* kh = k + (int64_t)head * k_head_stride + k_row0 * HD;
    const bf16_t* vh = vt + (int64_t)head * HD * vt_row_stride + k_row0;
    // K slot p holds chunk (p % CR) ^ kswz(key) of key p / CR, V^T slot p chunk (p % 4) ^ ((row >> 2) & 3) of channel p / 4
    auto load_tile = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < KCH / 64; ++i) {
        const int p = i * 64 + lane, row = p / CR;
        __builtin_amdgcn_global_load_lds((glb_void_t*)(kh + ((int64_t)tile * 32 + row) * HD + ((p % CR) ^ kswz<CR>(row)) * 8),
                                         (lds_void_t*)(mine + i * 64), 16, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < VCH / 64; ++i) {
        const int p = i * 64 + lane, row = p >> 2;
        __builtin_amdgcn_global_load_lds((glb_void_t*)(vh + row * vt_row_stride + (int64_t)tile * 32 + ((p & 3) ^ ((row >> 2) & 3)) * 8),
                                         (lds_void_t*)(mine + KCH + i * 64), 16, 0, 0);
      }
    };
    bf16x8 qf[KS];
    QuerySums qs;
    load_tile(wave);                                     // ahead: it is all that this wavefront may ever load
    request_queries<KS, HD>(q + (int64_t)head * q_head_stride, q0, lr, lg, S, qn, qs, qf);
    if (qn.ssq) scale_queries(qf, qs.factor<32>(qn, lg));
    f32x16 oacc[DT];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[d][r] = 0.f;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)mine;
    // MFMA row lr of a K tile is key swap23(lr): a lane's packed probabilities are then eight consecutive keys
    const int key = swap23(lr);
    const uint32_t krow = lds0 + (uint32_t)(key * CR) * 16, kx = (uint32_t)(lg ^ kswz<CR>(key)) * 16;
    const uint32_t vrow = lds0 + (uint32_t)(KCH + lr * 4) * 16, vx = (uint32_t)(lg ^ ((lr >> 2) & 3)) * 16;
    for (int t = wave; t < NT; t += 8) {
      vm_wait<0>();
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 kf[KS], vf[2][DT];
      static_for<KS>([&](auto i_) __attribute__((always_inline)) { constexpr int i = decltype(i_)::value; kf[i] = lds_read16<0>(krow + (kx ^ (uint32_t)(i * 32))); });
      static_for<2 * DT>([&](auto i_) __attribute__((always_inline)) {
        constexpr int u = decltype(i_)::value / DT, d = decltype(i_)::value % DT;
        vf[u][d] = lds_read16<d * 32 * 4 * 16>(vrow + (vx ^ (uint32_t)(u * 32)));
      });
      lds_wait<0>();
      __builtin_amdgcn_sched_barrier(0);
      if (t + 8 < NT) load_tile(t + 8);                  // the tile is in registers: its LDS is free
      const int valid = (int)(L - (int64_t)t * 32);      // >= 1; < 32 only in a ragged last tile
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
      // register r of lane group lg: key (r / 8) * 16 + lg * 8 + r % 8 of the tile
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = (r >> 3) * 16 + lg * 8 + (r & 7) < valid ? s[r] : -INFINITY;
        mx = fmaxf(mx, s[r]);
      }
      const float mn = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, 64)));
      const float ref = mn == -INFINITY ? 0.f : mn;      // nothing but scores of -inf so far: they weigh 0, not 2^(inf - inf)
      const float al = __builtin_amdgcn_exp2f(m - ref);  // 2^-inf = 0 at the first tile
      m = mn;
      l *= al;
      uint4 pf[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          w[j] = cvt_pk_bf16(__builtin_amdgcn_exp2f(s[u * 8 + 2 * j] - ref), __builtin_amdgcn_exp2f(s[u * 8 + 2 * j + 1] - ref));
          l = add_pk_bf16(w[j], l);
        }
        pf[u] = make_uint4(w[0], w[1], w[2], w[3]);
      }
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] *= al;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int d = 0; d < DT; ++d)
          oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u][d], __builtin_bit_cast(bf16x8, pf[u]), oacc[d], 0, 0, 0);
    }
    // partial results, unnormalised, fp32 [query][channel] in this wavefront's piece, 16-byte chunks XOR-swizzled with the query
    float4* o4 = (float4*)mine;
    constexpr int XO = HD / 4 - 1;
    const float lt = l + __shfl_xor(l, 32, 64);
    if (lg == 0) ml[wave][lr] = make_float2(m, lt);
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        o4[lr * (HD / 4) + ((d * 8 + g * 2 + lg) ^ (lr & XO))] = make_float4(oacc[d][g * 4], oacc[d][g * 4 + 1], oacc[d][g * 4 + 2], oacc[d][g * 4 + 3]);
  }
  __syncthreads();
  constexpr int TPQ = 512 / QB, C4 = HD / 4 / TPQ;       // threads per query, 4-channel chunks per thread, TPQ chunks apart
  const int ql = tid / TPQ, c0 = tid % TPQ;
  if (q0 + ql >= S) return;
  const float4* const o4 = (const float4*)smem + ql * (HD / 4);
  const int x0 = ql & (HD / 4 - 1);
  float mt = -INFINITY, lt = 0.f;
  float4 o[C4];
#pragma unroll
  for (int c = 0; c < C4; ++c) o[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  auto sum = [&](auto n_) __attribute__((always_inline)) {               // n > 0: all reads in flight together
    constexpr int n = decltype(n_)::value, U = n > 0 ? n : 1;
    const int np = n > 0 ? n : parts;
#pragma unroll U
    for (int w = 0; w < np; ++w) mt = fmaxf(mt, ml[w][ql].x);
#pragma unroll U
    for (int w = 0; w < np; ++w) {
      const float2 v = ml[w][ql];
      const float f = __builtin_amdgcn_exp2f(v.x - mt);
      lt += v.y * f;
#pragma unroll
      for (int c = 0; c < C4; ++c) {
        const float4 x = o4[w * MINE + ((c0 + c * TPQ) ^ x0)];
        o[c].x += x.x * f; o[c].y += x.y * f; o[c].z += x.z * f; o[c].w += x.w * f;
      }
    }
  };
  if (parts == 8) sum(std::integral_constant<int, 8>{}); else sum(std::integral_constant<int, 0>{});
  const float inv = 1.f / lt;
#pragma unroll
  for (int c = 0; c < C4; ++c)
    *(uint2*)(out + (q0 + ql) * ldo + (int64_t)head * HD + (c0 + c * TPQ) * 4) =
        make_uint2(cvt_pk_bf16(o[c].x * inv, o[c].y * inv), cvt_pk_bf16(o[c].z * inv, o[c].w * inv));
}

// Combines the key ranges of the split work ids: O = sum_i 2^(m_i - m) O_i / sum_i 2^(m_i - m) l_i with
// m = max_i m_i.  One thread per (query, 4 channels).  A block of 256 threads covers all channels of
// 256 / (HD/4) consecutive queries (query index fastest), so that partials are read in whole 128-byte
// lines and every output row is written from one block.
template <int HD, int QB>
__global__ __launch_bounds__(256) void k_attn_merge(const float* __restrict__ partial, int n_full, int n_tail,
                                                    int parts, int qblocks, int64_t S,
                                                    bf16_t* __restrict__ out, int64_t ldo) {
  constexpr int C4 = HD / 4, QPB = 256 / C4, SLOT = 2 * QB + QB * HD;
  const int tid = (int)threadIdx.x;
  const int gq = (int)blockIdx.x * QPB + tid % QPB;      // query index over all split work ids
  const int j = gq / QB, ql = gq % QB, c4 = tid / QPB;
  if (j >= n_tail) return;
  const int wid = n_full + j, head = wid / qblocks;
  const int64_t qi = (int64_t)(wid % qblocks) * QB + ql;
  if (qi >= S) return;
  const float* ps = partial + (size_t)j * parts * SLOT;
  float m = -INFINITY;
  for (int i = 0; i < parts; ++i) m = fmaxf(m, ps[(size_t)i * SLOT + ql]);
  float l = 0.f, o0 = 0.f, o1 = 0.f, o2 = 0.f, o3 = 0.f;
  for (int i = 0; i < parts; ++i) {
    const float* pi = ps + (size_t)i * SLOT;
    const float w = __builtin_amdgcn_exp2f(pi[ql] - m);
    const float4 v = *(const float4*)(pi + 2 * QB + ((size_t)c4 * QB + ql) * 4);
    l += w * pi[QB + ql];
    o0 += w * v.x; o1 += w * v.y; o2 += w * v.z; o3 += w * v.w;
  }
  const float inv = 1.f / l;
  uint2 pk;
  pk.x = cvt_pk_bf16(o0 * inv, o1 * inv);
  pk.y = cvt_pk_bf16(o2 * inv, o3 * inv);
  *(uint2*)(out + qi * ldo + (int64_t)head * HD + c4 * 4) = pk;
}

// partial results of at most 256 blocks of at most 256 queries
size_t attn_bf16_scratch_bytes(int d) { return (size_t)256 * (512 + 256 * (size_t)d) * sizeof(float); }

static constexpr int attn_slots(int qb, int kg) { return qb == 128 && kg < 2 ? 512 : 256; }   // blocks that the chip holds at once
// What a call takes: queries per block (32: k_attn_few), key groups, and key ranges that the work ids of the last round are cut into
struct AttnRoute { int qb, kg, parts; };
static AttnRoute attn_bf16_route(int64_t S, int64_t L, int h, int d, bool scratch) {
  // 256 queries per block share every K / V^T tile (half the LDS fill traffic per query) whenever that
  // still gives the grid half a round of blocks and the key range a few tiles; otherwise 128 queries per
  // block with the keys split over two groups, which halves the length of a block.
  const bool wide = L >= 256 && ((S + 255) / 256) * h >= 128;
  // Few enough blocks of 32 queries for one round (one to a CU at head_dim 128, two at 64) and at most eight tiles to a
  // wavefront: k_attn_few.  Beyond either line the other shapes are as fast (us): 1008 x 1680 x 16 heads of 64 (512 blocks) 17.9
  // against 20.3, 1000 x 1900 x 8 heads of 128 (256) 19.9 and 24.2, 700 x 1000 x 12 of 128 (264) 24.0 and 20.6, 100 x 3000 x 8 of 128
  // (32) 22.7 and 19.8.  Inside a stage, with the queries' row sums to read, heads of 64 meet earlier: 1008 x 1680 x 16 22.3 against
  // 21.6 (merge included), 1200 x 1600 x 12 21.1 and 20.8, 1200 x 1200 x 12 18.7 and 19.4, 672 x 1008 x 16 16.3 and 17.6; 1008 x 77 x 16
  // 9.3 and 10.2.
  const bool few = L <= 1920 && (S + 31) / 32 * h <= (d == 128 ? 256 : 512);
  // Few keys: a block's start and end weigh as much as its tiles, so blocks of four wavefronts, two to a CU, fill each other's
  // gaps.  Short key ranges, or up to 16 tiles where two rounds of such blocks are full (us): 6240 x 512 x 12 of 128 35.0 -> 31.5,
  // 1560 x 512 x 12 of 128 15.2 -> 13.4, 3000 x 1000 x 24 of 128 54.4 -> 50.6, 8000 x 200 x 16 of 64 17.7 -> 16.5; not at 3000 x 512 x
  // 16 of 64 (12.3 with 256 queries, 12.9) or 3000 x 1000 x 10 of 128 (22.9 with two groups, 34.2).
  const bool pairs = (L <= 512 && (d == 128 || !wide)) || (L <= 1024 && (S + 127) / 128 * h > 512);
  AttnRoute r{32, 8, 1};
  if (few) return r;
  r.qb = !pairs && wide ? 256 : 128;
  r.kg = pairs || wide ? 1 : 2;
  // One block (of 4 wavefronts: two) fits per compute unit, so the grid runs in rounds of `slots` blocks.  Whole rounds keep one
  // block per work id; the work ids left over for the last round are cut into key ranges (at least 8
  // key tiles each) so that the round is both shorter and wider, and a merge kernel joins the ranges.
  const int slots = attn_slots(r.qb, r.kg), W = (int)((S + r.qb - 1) / r.qb) * h, n_tail = W % slots, NKT = (int)((L + 63) / 64);
  if (n_tail > 0 && scratch) {
    r.parts = slots / n_tail;
    if (r.parts > 8) r.parts = 8;
    if (r.parts > NKT / 8) r.parts = NKT / 8;
    if (r.parts < 1) r.parts = 1;
  }
  return r;
}
// Whether blocks of eight wavefronts are k_attn_turns or k_attn_bf16.  Turns gain a few per cent of every tile and cost 1 to 3 us at a
// block's ends (the first tile in plain order, the halves half a turn apart, twice the tiles requested before the first product), so
// they take many tiles, and many blocks, whose ends overlap others' tiles only where there is more than a round.  Both inside a
// stage, on one card, k_attn_bf16 / k_attn_turns in us, queries x keys x heads of 128:
//   256 queries, less than a round of blocks: 2048 x 520 x 16 25.3 / 26.9, 1304 x 2000 x 24 57.7 / 59.0, 2560 x 3000 x 20 84.9 / 88.4,
//     x 5000 136.4 / 134.1, 2048 x 4000 x 16 (in two key ranges) 76.4 / 76.6, x 6000 103.0 / 100.8, but 3000 x 7600 x 14 183.0 / 184.7, 5504 x
//     8256 x 6 184 / 189: on a chip that is far from full the pinned order has clock to spare; at least one round: 4096 x 1100 x 16 46.3 / 46.7, x 2000 69.4 / 69.2,
//     x 2500 84.1 / 83.2, x 4500 137.8 / 134.4, 9000 x 1500 x 12 97.1 / 97.7, x 3000 169.4 / 167.3, x 9000 465 / 459, 6240 x 9360 x 12 327 / 321
//   two key groups: 1560 x 520 x 12 20.3 / 23.0, x 1000 25.9 / 27.8, x 2200 41.0 / 41.6, x 2500 45.3 / 44.9, x 4500 70.1 / 67.5; 3000
//     x 1500 x 10 35.5 / 35.9, x 2000 42.6 / 42.2, x 3000 57.0 / 55.2; in two key ranges 2000 x 2500 x 8 38.4 / 38.8, x 3500 45.3 / 45.1,
//     1304 x 3000 x 8 37.6 / 38.2, x 4500 47.3 / 47.1; in four 1000 x 2800 x 8 31.6 / 32.2
// Heads of 64 spend more of a tile on exponentials than on products, so a turn of the one is longer than of the other, and nothing is
// gained at any size: 2040 x 2040 x 32 43.4 / 44.3, 4096 x 9000 x 16 155 / 159, 14400 x 14400 x 16 889 / 910, 8000 x 20000 x 64 2514 / 2563; two key
// groups 2000 x 1500 x 12 22.2 / 23.1, 3000 x 9000 x 10 82.0 / 85.3.
static bool attn_bf16_turns(const AttnRoute& r, int64_t S, int64_t L, int h, int d) {
  const int64_t tiles = (L + 63) / 64, blocks = (S + r.qb - 1) / r.qb * h;
  if (d == 64) return false;
  if (r.qb == 256) return blocks >= 256 ? tiles >= 36 : blocks * r.parts >= 192 && tiles >= 80;
  return r.kg == 2 && tiles >= (r.parts > 1 ? 32 * r.parts : blocks >= 192 ? 32 : 38);
}
// for the tests, which state the kernel that each of their shapes is meant to reach
extern "C" void dp_attn_bf16_route(int64_t S, int64_t L, int32_t h, int32_t d, int32_t* queries_groups_ranges) {
  const AttnRoute r = attn_bf16_route(S, L, h, d, true);
  const int32_t v[3] = {r.qb, r.kg, r.parts};
  for (int i = 0; i < 3; ++i) queries_groups_ranges[i] = v[i];
}
extern "C" int dp_attn_bf16_turns(int64_t S, int64_t L, int32_t h, int32_t d) {
  return attn_bf16_turns(attn_bf16_route(S, L, h, d, true), S, L, h, d);
}

template <int HD, int QB, int KG, bool TURNS>
static void launch_attn_cfg(const bf16_t* q, int64_t q_head_stride, const bf16_t* k, int64_t k_head_stride,
                            int64_t k_row0, const bf16_t* vt, int64_t vt_row_stride, int64_t S, int64_t L,
                            int h, bf16_t* out, int64_t ldo, float* scratch, int parts, const AttnQNorm& qn, hipStream_t st) {
  constexpr int tile = (64 * (HD / 8) + HD * 8) * 16, lds = (TURNS ? 4 : 2 * KG) * tile, threads = QB * KG * 2;
  void (*const kernel)(const bf16_t*, int64_t, const bf16_t*, int64_t, int64_t, const bf16_t*, int64_t, int64_t, int64_t, bf16_t*, int64_t, int, int, int, int, float*, AttnQNorm) = [] {
    if constexpr (TURNS) return &k_attn_turns<HD, KG>; else return &k_attn_bf16<HD, QB / 32, KG>;
  }();
  const int qblocks = (int)((S + QB - 1) / QB);
  const int W = qblocks * h, n_tail = W % attn_slots(QB, KG), n_full = W - n_tail;
  dim3 grid((unsigned)(n_full + (n_tail * parts + 7) / 8 * 8));
  static std::atomic<uint64_t> done;
  allow_dynamic_lds((const void*)kernel, lds, done);
  kernel<<<grid, threads, lds, st>>>(q, q_head_stride, k, k_head_stride, k_row0, vt, vt_row_stride, S, L, out, ldo, qblocks, n_full, n_tail, parts, scratch, qn);
  if (parts > 1) {
    constexpr int QPB = 256 / (HD / 4);                  // queries per merge block
    k_attn_merge<HD, QB><<<(unsigned)(n_tail * (QB / QPB)), 256, 0, st>>>(scratch, n_full, n_tail, parts, qblocks, S, out, ldo);
  }
}

template <int HD>
static void launch_attn_few(const bf16_t* q, int64_t q_head_stride, const bf16_t* k, int64_t k_head_stride, int64_t k_row0,
                            const bf16_t* vt, int64_t vt_row_stride, int64_t S, int64_t L, int h, bf16_t* out, int64_t ldo,
                            const AttnQNorm& qn, hipStream_t st) {
  constexpr int QB = 32, tile = 2 * 32 * HD * 2, part = QB * HD * 4, lds = 8 * (tile > part ? tile : part);
  const int qblocks = (int)((S + QB - 1) / QB), n = qblocks * h;
  static std::atomic<uint64_t> done;
  allow_dynamic_lds((const void*)k_attn_few<HD>, lds, done);
  k_attn_few<HD><<<(unsigned)((n + 7) / 8 * 8), 512, lds, st>>>(q, q_head_stride, k, k_head_stride, k_row0, vt, vt_row_stride, S, L, out, ldo, qblocks, n, qn);
}

void launch_attn_bf16(const bf16_t* q, int64_t q_head_stride, const bf16_t* k, int64_t k_head_stride,
                      int64_t k_row0, const bf16_t* vt, int64_t vt_row_stride, int64_t S, int64_t L,
                      int h, int d, bf16_t* out, int64_t ldo, float* scratch, const AttnQNorm* qnorm, hipStream_t st) {
  if (S <= 0 || L <= 0) return;
  const AttnQNorm qn = qnorm ? *qnorm : AttnQNorm{nullptr, 0, 0, 0.f, 0.f, 0.f};
  AttnRoute r = attn_bf16_route(S, L, h, d, scratch != nullptr);
  // The larger blocks reach a head's rows of V^T by 32-bit offsets from its first: signed, in elements, or unsigned, in bytes.  Key
  // buffers too long for that (2^24 positions of 128 channels, whatever this call reads of them) take the kernel that has 64.
  if ((int64_t)d * vt_row_stride > (int64_t)1 << 31) r = AttnRoute{32, 8, 1};
  const bool turns = attn_bf16_turns(r, S, L, h, d);
#define ATTN_ARGS q, q_head_stride, k, k_head_stride, k_row0, vt, vt_row_stride, S, L, h, out, ldo
#define ATTN_CASE(HD) do { \
    if (r.qb == 32) launch_attn_few<HD>(ATTN_ARGS, qn, st); \
    else if (r.qb == 256 && HD == 128 && turns) launch_attn_cfg<128, 256, 1, true>(ATTN_ARGS, scratch, r.parts, qn, st); \
    else if (r.qb == 256) launch_attn_cfg<HD, 256, 1, false>(ATTN_ARGS, scratch, r.parts, qn, st); \
    else if (r.kg == 1) launch_attn_cfg<HD, 128, 1, false>(ATTN_ARGS, scratch, r.parts, qn, st); \
    else if (HD == 128 && turns) launch_attn_cfg<128, 128, 2, true>(ATTN_ARGS, scratch, r.parts, qn, st); \
    else launch_attn_cfg<HD, 128, 2, false>(ATTN_ARGS, scratch, r.parts, qn, st); \
  } while (0)
  if (d == 128) ATTN_CASE(128); else ATTN_CASE(64);
#undef ATTN_CASE
#undef ATTN_ARGS
}
