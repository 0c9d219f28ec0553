// Tree-masked attention on the matrix cores (Sec. 2.1 attention, Sec. 2.2 and 3.3.2
// tree mask), bf16, d_head = 128, grouped-query.
//
// A workgroup of eight waves owns one (request, KV head, block of query rows, chunk of
// cache slots).  Its waves cut the chunk into eight runs of 32-slot tiles; each wave
// streams the K and V rows of its run from HBM exactly once for all query rows of the
// block (the g query heads of the group times the tree nodes), keeps an online softmax,
// and the eight states are folded together through LDS.  (Blocks of 64 query rows: four runs,
// whose tiles two waves share.)  If the request's whole cache
// range is one chunk the block's output is final; otherwise an un-normalised partial
// (running max, sum, output) is left per query row and a second kernel merges the chunks.
// The committed context is visible to every node; a tree slot is visible to a node iff its
// bit is set in the node's ancestor mask.
//
// MFMA use (v_mfma_f32_16x16x32_bf16, D[4*(l/16)+i][l%16]):
//   S^T = K Q^T : A = 16 slots x 32 d (16 B per lane, read from an LDS copy of the K tile),
//                 B = 32 d x 16 query rows (registers, loaded once).
//   O^T = V^T P^T: B = P^T is exactly the S^T registers of two 16-slot tiles (the
//                 contraction order over the 32 slots is free, so no shuffle is
//                 needed); A = V^T needs 8 slots per lane for one d: two transposing reads
//                 (ds_read_b64_tr_b16) of an LDS copy of the V tile.
//
// What bounds it: with few query rows the K/V stream from HBM; with many (the tiles then come out of L2) the instructions of a
// tile, two waves per SIMD.  There the way of a tile through registers to LDS was the largest part (70B shape, 128 rows behind
// 4096 slots, 43.7 us alone: 36.9 without the global loads, 23.6 without them and the LDS stores), and the V fragments came in
// 32-bit reads with a permutation each.  Direct-to-LDS loads and transposing reads: 48.1 -> 38.0 us in the step, one request of
// a few rows behind 32768 slots 27.3 -> 26.1 us.
#include "sp_launch.h"

#define DH 128
#define TILE_BYTES (32 * 256)   // 32 slots of K or V

struct AttnArgs {
  const bf16_t* q;          // [M][n_q][DH]
  const ReqTables* tables;
  KvGeom g;
  int layer, n_q, n_kv;
  float* part_o;            // [units][DH], followed by [units][2] (running max, sum)
  bf16_t* out;              // rows of n_q * DH columns, in fragment order or (frag false) row-major
  bool frag;
  const AttnPlan* plan;     // device copy of the call's plan (written by the kernel that opens the forward)
};

// Online softmax of a wave over QT tiles of 16 query rows.  mrun is the running maximum of the raw scores q.k; negm =
// -mrun*sc (0 while mrun is -inf), so that exp2(fma(s, sc, negm)) is the softmax weight.
template <int QT>
struct AttnState {
  f32x4_t o[QT][8];
  float mrun[QT], lrun[QT], negm[QT];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      mrun[t] = -INFINITY; lrun[t] = 0.f; negm[t] = 0.f;
#pragma unroll
      for (int d = 0; d < 8; ++d) o[t][d] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    }
  }
};
#define ATTN_SC (0.08838834764831845f * 1.4426950408889634f)   // 1/sqrt(128) * log2(e)

// A tile's rows lie in LDS as they do in memory, 256 bytes each, but that the 16-byte units of a row are exchanged by the row's
// number (unit u is at place u ^ unit_swap(row)): the direct-to-LDS loads leave no room for padding.  Sixteen rows' fragments
// of the same columns then lie in sixteen different units, and so do the four rows x four units that sixteen lanes of a
// transposing read ask for: two neighbouring rows differ in the upper two bits of the unit.
__device__ __forceinline__ int unit_swap(int row) { return (row & 3) * 4 + ((row >> 2) & 3); }

// Scores of a 32-slot tile; ka: the lane's places of its K fragments, row l15 of each 16-slot half, 16 B at d = s*32 + kg*8.
template <int QT>
__device__ __forceinline__ void attn_scores(f32x4_t (&sacc)[QT][2], const u32x4_t (&qf)[QT][4], const char* kt, const int (&ka)[4]) {
#pragma unroll
  for (int t = 0; t < QT; ++t)
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) sacc[t][t2] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x4_t kf = *reinterpret_cast<const u32x4_t*>(kt + ka[s] + t2 * 4096);
#pragma unroll
      for (int t = 0; t < QT; ++t)
        sacc[t][t2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(&kf),
                                                              *reinterpret_cast<const bf16x8_t*>(&qf[t][s]),
                                                              sacc[t][t2], 0, 0, 0);
    }
}

// Scores of the tile with first slot s0, of a run that ends at w1, to weights (bf16 pairs, in the order of sacc's slots).
template <int QT>
__device__ __forceinline__ void attn_softmax(AttnState<QT>& st, const f32x4_t (&sacc)[QT][2], uint32_t (&pb)[QT][4],
                                             const unsigned long long (&anc)[QT][SP_W], int s0, int w1, int P, int span, int kg) {
  const float sc = ATTN_SC;
  const bool tail = s0 + 32 > P || s0 + 32 > w1;   // tile touches the tree region or the run's end
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float sv[8];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[t2 * 4 + i] = sacc[t][t2][i];
    if (tail) {
      // bits [n0, n0+64) of the row's 256-bit ancestor mask, n0 = first tree index of the tile
      const int n0 = s0 - P;
      unsigned long long win = 0ull;
#pragma unroll
      for (int w = 0; w < SP_W; ++w) {
        const int sh = w * 64 - n0;
        if (sh > -64 && sh < 64) win |= sh >= 0 ? (anc[t][w] << sh) : (anc[t][w] >> (-sh));
      }
      const int lim = w1 - s0, pfx = P - s0, tl = span - s0;   // offsets below: in run / committed / live
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int off = (j >> 2) * 16 + kg * 4 + (j & 3);
        const bool vis = (off < lim) & ((off < pfx) | ((off < tl) & (bool)((win >> off) & 1ull)));
        sv[j] = vis ? sv[j] : -INFINITY;
      }
    }
    float mx = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
    // The running maximum only has to bound the scores, so it is raised (and the
    // accumulators rescaled) only when some lane of the wave sees a larger score.
    if (__builtin_amdgcn_ballot_w64(mx > st.mrun[t])) {
      mx = quad_rows_max(mx);
      const float mnew = fmaxf(st.mrun[t], mx);
      const float alpha = (mnew == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f((st.mrun[t] - mnew) * sc);  // 0 from -inf
      st.lrun[t] *= alpha;
#pragma unroll
      for (int d = 0; d < 8; ++d) st.o[t][d] *= alpha;
      st.mrun[t] = mnew;
      st.negm[t] = (mnew == -INFINITY) ? 0.f : -mnew * sc;
    }
    float pv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) pv[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[j], sc, st.negm[t]));
    st.lrun[t] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
#pragma unroll
    for (int j = 0; j < 4; ++j) pb[t][j] = pack_bf16x2(pv[2 * j], pv[2 * j + 1]);
  }

}

// O^T += V^T P^T; va: the lane's places for the transposing reads.  Sixteen lanes read four slots x 16 columns, lane 4c + x of
// them gets the four slots of column G*32 + 8c + 4e + x, and so a lane's products of e = 0 and 1 are eight columns in a row.
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
__device__ __forceinline__ uint2 read_transposed(const char* p) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p)));
#else
  return uint2{0u, 0u};
#endif
}
template <int QT>
__device__ __forceinline__ void attn_pv(AttnState<QT>& st, const uint32_t (&pb)[QT][4], const char* vt, const int (&va)[4]) {
#pragma unroll
  for (int G = 0; G < 4; ++G)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint2 lo = read_transposed(vt + va[G] + e * 8), hi = read_transposed(vt + va[G] + e * 8 + 4096);
      const u32x4_t vf = {lo.x, lo.y, hi.x, hi.y};
#pragma unroll
      for (int t = 0; t < QT; ++t)
        st.o[t][2 * G + e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(&vf),
                                                                  *reinterpret_cast<const bf16x8_t*>(&pb[t][0]),
                                                                  st.o[t][2 * G + e], 0, 0, 0);
    }
}

// RQ groups of waves with QT tiles of 16 query rows each; the groups share the tiles that they bring in together.
// NT: every request of the call has a single block of query rows, so each K/V row is read by one workgroup only; the loads
// then carry the non-temporal hint and the rows pass through the caches without staying.
// K and V rows come in as whole 256-byte rows (a load instruction covers four), straight to an LDS tile of the wave, or (REGS)
// through registers, in which the next tile waits while this one is used.
#define AW 8              // waves per workgroup
template <int RQ, int QT, bool PAGED, bool NT, bool REGS>
__global__ void __launch_bounds__(64 * AW) k_attn_bf16(AttnArgs a) {
  constexpr int SR = AW / RQ;                      // runs of slots
  const AttnPlan& plan = *a.plan;
  // K and V tiles of the eight waves (RQ > 1: two sets of tiles) in arrays of their own, so that the compiler knows which loads
  // a read has to wait for; the same bytes later carry the states being folded, query tile 0's and 1's.
  static_assert(AW * TILE_BYTES == AW * 8 * 64 * 16 && QT <= 2, "a query tile's states fill an array");
  __shared__ __attribute__((aligned(16))) char s_k[AW * TILE_BYTES];
  __shared__ __attribute__((aligned(16))) char s_v[AW * TILE_BYTES];
  __shared__ float s_m[AW][QT * 16];
  __shared__ float s_l[AW][QT * 16];

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  // KV head fastest: consecutive workgroup ids go round-robin over the 8 XCDs, so all query
  // blocks and chunks of one KV head share one XCD's L2 and its K/V rows are fetched from HBM once
  // (uni: quotients come out of vector registers; what the tiles' buffers are built from has to be scalar)
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  const int item = uni(blockIdx.x / a.n_kv);
  const int kvh = blockIdx.x - item * a.n_kv;
  // Segment 0's fields are asked for together with the segment count: a call with one request (the rule) then
  // waits for one round trip to the plan, not for two in a row.
  int sg_item0 = plan.seg_item0[0], sg_chunks = plan.seg_chunks[0], sg_rows = plan.seg_rows[0], sg_row0 = plan.seg_row0[0];
  int sg_P = plan.seg_P[0], sg_T = plan.seg_T[0], sg_clen = plan.seg_clen[0], sg_req = plan.seg_req[0];
  int sg_first = plan.seg_first[0], sg_unit0 = plan.seg_unit0[0];
  long long sg_base = plan.seg_base[0];
  const int n_seg = plan.n_seg, units_total = plan.units_total;
  if (n_seg > 1) {
    // each lane looks at a segment
    static_assert(SP_BATCH == 64, "one lane per segment");
    const int seg = uni(__popcll(__builtin_amdgcn_ballot_w64(lane < n_seg && item >= plan.seg_item0[lane])) - 1);
    sg_item0 = plan.seg_item0[seg]; sg_chunks = plan.seg_chunks[seg]; sg_rows = plan.seg_rows[seg];
    sg_row0 = plan.seg_row0[seg]; sg_P = plan.seg_P[seg]; sg_T = plan.seg_T[seg]; sg_clen = plan.seg_clen[seg];
    sg_req = plan.seg_req[seg]; sg_first = plan.seg_first[seg]; sg_unit0 = plan.seg_unit0[seg];
    sg_base = plan.seg_base[seg];
  }
  const int local = item - sg_item0;
  const int chunks = sg_chunks;
  const int qb = uni(local / chunks), ch = local - qb * chunks;
  const int g = a.n_q / a.n_kv;
  const float inv_g = 1.f / (float)g;              // (qi + 0.5) * inv_g truncates to qi / g for these small integers
  const int seg_rows = sg_rows, row0 = sg_row0;
  const int nqrows = seg_rows * g;                 // query rows of this (request, KV head)
  const int P = sg_P, T = sg_T;
  const int span = P + T;
  const int c0 = ch * sg_clen;
  const int c1 = min(c0 + sg_clen, span);
  // this wave's run of 32-slot tiles inside [c0, c1)
  const int ntiles = (c1 - c0 + 31) >> 5;
  const int run = wave / RQ, group = wave % RQ;
  const int w0 = c0 + 32 * ((run * ntiles) / SR);
  const int w1 = min(c0 + 32 * (((run + 1) * ntiles) / SR), c1);
  const int l15 = lane & 15, kg = lane >> 4;

  // contiguous cache: the request's range starts at its base slot; paged: logical slots go through
  // the request's page table, one lookup per 32-slot tile (a tile never straddles a page)
  const size_t base_b = PAGED ? 0 : (size_t)sg_base * 256;
  const char* kplane = a.g.kv + ((size_t)(a.layer * 2 + 0) * a.n_kv + kvh) * a.g.plane_bytes + base_b;
  const char* vplane = a.g.kv + ((size_t)(a.layer * 2 + 1) * a.n_kv + kvh) * a.g.plane_bytes + base_b;
  // (read through the scalar cache: a lookup among the vector loads would wait for all of those before it)
  typedef const __attribute__((address_space(4))) int* const_int_p;
  const const_int_p pt = PAGED ? (const_int_p)(uintptr_t)(a.g.page_table + (size_t)uni(sg_req) * a.g.pt_stride) : nullptr;
  const int pg_sh = PAGED ? a.g.pg_shift : 0, pg_mask = (1 << pg_sh) - 1;
  // Loads of one 32-slot tile.  The tile is a buffer of its own, as long as its rows inside the request's data: rows behind
  // them come back as zeros without a memory access (and are masked later).
  unsigned lofs[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = (group * (8 / RQ) + i) * 4 + kg;
    lofs[i] = row * 256 + (l15 ^ unit_swap(row)) * 16;
  }
  // physical slot of a tile's first slot (a tile past the data: no rows of slot 0's)
  auto tile_slot = [&](int s0) -> size_t {
    const int t0 = uni(s0 < span ? s0 : 0);
    return PAGED ? ((size_t)pt[t0 >> pg_sh] << pg_sh) + (t0 & pg_mask) : (size_t)t0;
  };
#define SP_TILE_BUFFER(PLANE, S0, SLOT)                                                            \
    const auto buf_ = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(PLANE) + (SLOT) * 256, (short)0, \
                                                        uni(max(0, min(32, span - (S0)))) * 256, 0x00020000);
#define SP_LOAD_ROWS(DST, PLANE, S0, SLOT)                                                         \
  {                                                                                                \
    SP_TILE_BUFFER(PLANE, S0, SLOT)                                                                \
    _Pragma("unroll") for (int i = 0; i < 8 / RQ; ++i) load_to_lds<NT>(buf_, DST + i * 1024, lofs[i], 0); \
    __builtin_amdgcn_sched_barrier(0);                                                             \
  }
#define SP_FETCH_ROWS(DST, PLANE, S0, SLOT)                                                        \
  {                                                                                                \
    SP_TILE_BUFFER(PLANE, S0, SLOT)                                                                \
    _Pragma("unroll") for (int i = 0; i < 8; ++i) DST[i] = __builtin_amdgcn_raw_buffer_load_b128(buf_, lofs[i], 0, NT ? 2 : 0); \
  }

  // the first tile's loads go out before anything else that has to wait
  u32x4_t kreg[REGS ? 8 : 1], vreg[REGS ? 8 : 1];
  char* kt = s_k + wave * TILE_BYTES;
  char* vt = s_v + wave * TILE_BYTES;
  // tiles of a run that RQ waves share: two of them, K and V one behind the other; a wave brings in its part of the rows
  const int first = w0 < w1 ? w0 : span;
  const size_t first_slot = tile_slot(first);
  const int pair = run * 2 * TILE_BYTES, part = pair + group * (TILE_BYTES / RQ);
  if constexpr (RQ > 1) {
    SP_LOAD_ROWS(s_k + part, kplane, first, first_slot)
    SP_LOAD_ROWS(s_k + part + TILE_BYTES, vplane, first, first_slot)
  } else if constexpr (REGS) {
    SP_FETCH_ROWS(kreg, kplane, first, first_slot)
    SP_FETCH_ROWS(vreg, vplane, first, first_slot)
  } else {
    SP_LOAD_ROWS(kt, kplane, first, first_slot)
    SP_LOAD_ROWS(vt, vplane, first, first_slot)
  }

  // ---- query fragments and ancestor masks of this lane's query row per tile ------
  u32x4_t qf[QT][4];
  unsigned long long anc[QT][SP_W];
  const ReqTables* tab = a.tables + sg_req;
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int qi = (qb * RQ + group) * (QT * 16) + t * 16 + l15;  // index inside (request, KV head): node_local * g + gq
    const bool ok = qi < nqrows;
    const int nl = ok ? (int)(((float)qi + 0.5f) * inv_g) : 0, gq = ok ? qi - nl * g : 0;
    const bf16_t* qp = a.q + ((size_t)(row0 + nl) * a.n_q + (size_t)kvh * g + gq) * DH + kg * 8;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(qp + s * 32);
      qf[t][s] = ok ? v : (u32x4_t){0u, 0u, 0u, 0u};
    }
    const int node = sg_first + nl;
#pragma unroll
    for (int w = 0; w < SP_W; ++w) {
      const unsigned long long v = tab->anc[node][w];
      anc[t][w] = ok ? v : 0ull;
    }
  }

  AttnState<QT> st;
  st.init();

  int ka[4], va[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int vr = kg * 4 + (l15 >> 2);            // row of the lane's transposing reads in a 16-slot half
    ka[i] = l15 * 256 + ((i * 4 + kg) ^ unit_swap(l15)) * 16;
    va[i] = vr * 256 + ((i * 4 + (l15 & 3)) ^ unit_swap(vr)) * 16;
  }
  // no read of a tile may still be on its way when the loads that take its place go out
  auto reads_done = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
  auto loads_done_but_8 = [] { SP_WAIT_VMEM(8); asm volatile("" ::: "memory"); __builtin_amdgcn_sched_barrier(0); };
  if constexpr (RQ > 1) {
    // One barrier a tile: behind it the tile is there whole and nobody reads the other one any more.  Runs differ by a tile at
    // most; a wave that has none left goes on bringing up the barriers.
#define SP_SHARED_TILE(CUR, OTHER, S0)                                                             \
    if (it < steps) {                                                                              \
      const int s0 = (S0), nxt = s0 + 32 < w1 ? s0 + 32 : span;                                    \
      const size_t nxt_slot = tile_slot(nxt);                                                      \
      SP_WAIT_VMEM(0);                                                                             \
      reads_done();                                                                                \
      bare_barrier();                                                                              \
      SP_LOAD_ROWS(OTHER + part, kplane, nxt, nxt_slot)                                            \
      SP_LOAD_ROWS(OTHER + part + TILE_BYTES, vplane, nxt, nxt_slot)                               \
      if (s0 < w1) {                                                                               \
        f32x4_t sacc[QT][2];                                                                       \
        uint32_t pb[QT][4];                                                                        \
        attn_scores<QT>(sacc, qf, CUR + pair, ka);                                                 \
        attn_softmax<QT>(st, sacc, pb, anc, s0, w1, P, span, kg);                                  \
        attn_pv<QT>(st, pb, CUR + pair + TILE_BYTES, va);                                          \
      }                                                                                            \
      ++it;                                                                                        \
    }
    const int steps = (ntiles + SR - 1) / SR;
    for (int it = 0; it < steps;) {
      SP_SHARED_TILE(s_k, s_v, w0 + it * 32)
      SP_SHARED_TILE(s_v, s_k, w0 + it * 32)
    }
#undef SP_SHARED_TILE
  } else for (int s0 = w0; s0 < w1; s0 += 32) {
    // A tile's K rows make room for the next tile's as soon as its scores are there, its V rows behind the PV product; what
    // is waited for is the older half of the loads in flight.
    const int nxt = (s0 + 32 < w1) ? s0 + 32 : span;       // span: no rows
    const size_t nxt_slot = tile_slot(nxt);
    f32x4_t sacc[QT][2];
    uint32_t pb[QT][4];
    if constexpr (REGS) {
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4_t*>(vt + i * 1024 + lane * 16) = vreg[i];
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4_t*>(kt + i * 1024 + lane * 16) = kreg[i];
      __builtin_amdgcn_wave_barrier();
      SP_FETCH_ROWS(kreg, kplane, nxt, nxt_slot)
      SP_FETCH_ROWS(vreg, vplane, nxt, nxt_slot)
      attn_scores<QT>(sacc, qf, kt, ka);
      attn_softmax<QT>(st, sacc, pb, anc, s0, w1, P, span, kg);
      __builtin_amdgcn_wave_barrier();
      attn_pv<QT>(st, pb, vt, va);
      __builtin_amdgcn_wave_barrier();
    } else {
      loads_done_but_8();
      attn_scores<QT>(sacc, qf, kt, ka);
      reads_done();
      SP_LOAD_ROWS(kt, kplane, nxt, nxt_slot)
      attn_softmax<QT>(st, sacc, pb, anc, s0, w1, P, span, kg);
      loads_done_but_8();
      attn_pv<QT>(st, pb, vt, va);
      reads_done();
      SP_LOAD_ROWS(vt, vplane, nxt, nxt_slot)
    }
  }
  SP_WAIT_VMEM(0);
#undef SP_FETCH_ROWS
#undef SP_LOAD_ROWS
#undef SP_TILE_BUFFER

  // ---- fold the eight wave states (fixed order, so results do not depend on timing) ----
  // Every wave rescales its state to the common maximum and leaves it in LDS; after one barrier the block's
  // 4 * QT pieces (query tile t, 32 output columns G) are each summed over the waves with these query rows and written by
  // one of them.
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    st.lrun[t] = quad_rows_sum(st.lrun[t]);
    st.mrun[t] = st.mrun[t] * ATTN_SC;              // to the log2 domain (-inf stays -inf)
    if (kg == 0) s_m[wave][t * 16 + l15] = st.mrun[t];
  }
  __syncthreads();                       // every wave is done with its tiles; maxima are posted
  float mall[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < SR; ++w) m = fmaxf(m, s_m[w * RQ + group][t * 16 + l15]);
    mall[t] = m;
    const float f = (st.mrun[t] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(st.mrun[t] - m);
#pragma unroll
    for (int d = 0; d < 8; ++d) reinterpret_cast<f32x4_t*>(t == 0 ? s_k : s_v)[(wave * 8 + d) * 64 + lane] = st.o[t][d] * f;
    if (kg == 0) s_l[wave][t * 16 + l15] = st.lrun[t] * f;
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < (4 * QT + SR - 1) / SR; ++p) {
    const int piece = run + p * SR, t = piece >> 2, G = piece & 3;          // a piece of the wave's own query rows
    if (piece >= 4 * QT) break;
    const f32x4_t* fold = reinterpret_cast<const f32x4_t*>(t == 0 ? s_k : s_v);
    f32x4_t e0 = {0.f, 0.f, 0.f, 0.f}, e1 = {0.f, 0.f, 0.f, 0.f};
    float lsum = 0.f;
#pragma unroll
    for (int w = 0; w < SR; ++w) {
      e0 += fold[((w * RQ + group) * 8 + 2 * G) * 64 + lane];
      e1 += fold[((w * RQ + group) * 8 + 2 * G + 1) * 64 + lane];
      lsum += s_l[w * RQ + group][t * 16 + l15];
    }

    // e0[i] / e1[i] are output columns G*32 + 8*kg + i and + 4 of query row t*16 + l15.
    const int qi = (qb * RQ + group) * (QT * 16) + t * 16 + l15;
    if (qi >= nqrows) continue;
    const int nl = (int)(((float)qi + 0.5f) * inv_g), gq = qi - nl * g;
    const int head = kvh * g + gq;
    if (chunks == 1) {
      const float inv = 1.f / lsum;
      u32x4_t pk;
      pk.x = pack_bf16x2(e0[0] * inv, e0[1] * inv);
      pk.y = pack_bf16x2(e0[2] * inv, e0[3] * inv);
      pk.z = pack_bf16x2(e1[0] * inv, e1[1] * inv);
      pk.w = pack_bf16x2(e1[2] * inv, e1[3] * inv);
      *reinterpret_cast<u32x4_t*>(a.out + row_at(a.frag, row0 + nl, head * DH + G * 32 + 8 * kg, a.n_q * DH)) = pk;
    } else {
      const size_t unit = (size_t)sg_unit0 + (size_t)ch * seg_rows * a.n_q + (size_t)nl * a.n_q + head;
      float* po = a.part_o + unit * DH;
      *reinterpret_cast<f32x4_t*>(po + G * 32 + 8 * kg) = e0;
      *reinterpret_cast<f32x4_t*>(po + G * 32 + 8 * kg + 4) = e1;
      if (G == 0 && kg == 0) {
        float* part_ml = a.part_o + (size_t)units_total * DH;
        // the common maximum of query row t*16 + l15 (a wave-uniform choice between the two tiles' registers)
        const float m_t = (t == 0) ? mall[0] : mall[QT - 1];
        part_ml[unit * 2] = m_t; part_ml[unit * 2 + 1] = lsum;
      }
    }
  }
}

// One wave per (row, query head) of the requests that were cut into several chunks: combine the
// chunk partials (log2-domain maxima).  Lane c first takes chunk c's (max, sum) and turns them into
// the chunk's weight; the outputs are then accumulated chunk by chunk, two columns per lane.
__global__ void __launch_bounds__(256) k_attn_merge(AttnArgs a, int M) {
  const AttnPlan& plan = *a.plan;
  int sg_chunks = plan.seg_chunks[0], sg_rows = plan.seg_rows[0], sg_unit0 = plan.seg_unit0[0], sg_row0 = plan.seg_row0[0];
  const int n_seg = plan.n_seg;
  const float* part_ml = a.part_o + (size_t)plan.units_total * DH;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // a workgroup takes four rows of a head; the two that fill the output's 128-byte lines (eight rows in fragment order)
  // run on the same XCD, whose L2 puts the lines together
  const int pair = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7), row8 = pair / a.n_q, head = pair - row8 * a.n_q;
  const int row = row8 * 8 + ((blockIdx.x >> 3) & 1) * 4 + wave;
  if (row >= M) return;
  if (n_seg > 1) {                       // each lane looks at a segment
    const int first = plan.seg_row0[lane], seg = __ffsll((unsigned long long)__builtin_amdgcn_ballot_w64(lane < n_seg && row >= first && row < first + plan.seg_rows[lane])) - 1;
    sg_chunks = plan.seg_chunks[seg]; sg_rows = plan.seg_rows[seg]; sg_unit0 = plan.seg_unit0[seg]; sg_row0 = plan.seg_row0[seg];
  }
  const int chunks = sg_chunks, seg_rows = sg_rows;
  if (chunks == 1) return;               // written directly by the attention kernel
  const size_t stride = (size_t)seg_rows * a.n_q;
  const size_t u0 = (size_t)sg_unit0 + (size_t)(row - sg_row0) * a.n_q + head;
  float acc0 = 0.f, acc1 = 0.f, lsum = 0.f, mx = -INFINITY;
  for (int c0 = 0; c0 < chunks; c0 += 64) {        // blocks of 64 chunks (one is the rule)
    const int c = c0 + lane;
    float m = -INFINITY, l = 0.f;
    if (c < chunks) {
      const float2 ml = *reinterpret_cast<const float2*>(part_ml + (u0 + c * stride) * 2);
      m = ml.x; l = ml.y;
    }
    const float bm = wave_max(m);
    const float nmx = fmaxf(mx, bm);
    if (nmx == -INFINITY) continue;
    const float resc = (mx == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mx - nmx);
    acc0 *= resc; acc1 *= resc; lsum *= resc;
    mx = nmx;
    const float wgt = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mx);
    lsum += wave_sum(wgt * l);
    const int nb = min(64, chunks - c0);
    int j = 0;
    // sixteen chunks' partial rows in flight at a time: the loop is a chain of memory round trips otherwise
    for (; j + 16 <= nb; j += 16) {
      float o0[16], o1[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float* po = a.part_o + (u0 + (size_t)(c0 + j + i) * stride) * DH;
        const float2 v = *reinterpret_cast<const float2*>(po + 2 * lane);
        o0[i] = v.x; o1[i] = v.y;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float w1 = __shfl(wgt, j + i, 64);
        acc0 += w1 * o0[i]; acc1 += w1 * o1[i];
      }
    }
    for (; j + 4 <= nb; j += 4) {
      float w4[4], o0[4], o1[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        w4[i] = __shfl(wgt, j + i, 64);
        const float* po = a.part_o + (u0 + (size_t)(c0 + j + i) * stride) * DH;
        const float2 v = *reinterpret_cast<const float2*>(po + 2 * lane);
        o0[i] = v.x; o1[i] = v.y;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) { acc0 += w4[i] * o0[i]; acc1 += w4[i] * o1[i]; }
    }
    for (; j < nb; ++j) {
      const float w1 = __shfl(wgt, j, 64);
      const float2 v = *reinterpret_cast<const float2*>(a.part_o + (u0 + (size_t)(c0 + j) * stride) * DH + 2 * lane);
      acc0 += w1 * v.x; acc1 += w1 * v.y;
    }
  }
  const float inv = 1.f / lsum;
  *reinterpret_cast<uint32_t*>(a.out + row_at(a.frag, row, head * DH + 2 * lane, a.n_q * DH)) = pack_bf16x2(acc0 * inv, acc1 * inv);
}

hipError_t sp_launch_attn_bf16(const bf16_t* q, const ReqTables* tables, KvGeom g, int layer, const AttnPlan& plan,
                               const AttnPlan* plan_dev, float* part, bf16_t* out, bool frag, int M,
                               int n_q, int n_kv, int d_head, hipStream_t st) {
  if (d_head != DH || g.row_bytes != 256) return hipErrorInvalidValue;
  AttnArgs a;
  a.q = q; a.tables = tables; a.g = g; a.layer = layer; a.n_q = n_q; a.n_kv = n_kv;
  a.part_o = part;
  a.out = out;
  a.frag = frag;
  a.plan = plan_dev;
  dim3 grid(plan.total_items * n_kv);
#define SP_ATTN_GO(RQV, QTV, PG, NTV, REGSV) hipLaunchKernelGGL((k_attn_bf16<RQV, QTV, PG, NTV, REGSV>), grid, dim3(64 * AW), 0, st, a)
#define SP_ATTN_PG(RQV, QTV, PG) \
  { if (RQV > 1 || plan.loads == ATTN_SHARED) SP_ATTN_GO(RQV, QTV, PG, false, false); else if (plan.loads == ATTN_STREAM_REGS) SP_ATTN_GO(1, QTV, PG, true, true); else SP_ATTN_GO(1, QTV, PG, true, false); }
#define SP_ATTN_QT(RQV, QTV) { if (g.page_table) SP_ATTN_PG(RQV, QTV, true) else SP_ATTN_PG(RQV, QTV, false) }
  switch (plan.qt) {
    case 1: SP_ATTN_QT(1, 1) break;
    case 2: SP_ATTN_QT(1, 2) break;
    case 4: SP_ATTN_QT(2, 2) break;
    default: return hipErrorInvalidValue;
  }
#undef SP_ATTN_QT
#undef SP_ATTN_PG
#undef SP_ATTN_GO
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !plan.any_split) return e;
  hipLaunchKernelGGL(k_attn_merge, dim3(((M + 7) / 8 * n_q + 7) / 8 * 16), dim3(256), 0, st, a, M);
  return hipGetLastError();
}
