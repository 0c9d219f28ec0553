// bf16 projections for many rows (plain products from 161 rows on, gate/up from 129 or, where sp_gemm_mid.hip takes it,
// 161 or 193: a cold ragged batch forwards several hundred tree nodes at once, Sec. 4 "Implementation" / Sec. 4.4).  Here the
// matrix cores, not the weight stream, set the pace, so each wave keeps SPW strips of 16 weight rows in registers and every
// activation fragment it reads from LDS feeds SPW MFMAs.  Two kernels: k_gemm_wide here, over row-major weights in blocks of
// 128 rows and, from 385 on, 256, and over weights in fragment order in blocks of 128 up to 384 rows (gate/up 256, or 320
// where either kernel makes one round of workgroups); k_gemm_wide32 further down beyond those.  A workgroup covers up to 16*MT rows x
// 64*SPW output columns.  Full row blocks come first in launch order, and those of one column
// tile get consecutive ids modulo 8: they run at the same time on the same XCD and share the
// tile's weights through its L2.  The last, partial row block of every tile comes after all
// full ones and runs a body compiled for its own height, so the short workgroups fill the CUs
// that the full ones leave over.
//
//   out[y][m][n] = sum_{k in slice y} X[m][k] * W[n][k]        (f32 partial sums)
//   gate/up:      act[m][f] = silu(X Wg^T) * (X Wu^T)          (each wave pairs gate and up strips)
#include "sp_launch.h"

#ifndef WKC
#define WKC 64                  // k per staged chunk
#endif
#define WXS (WKC * 2 + 16)      // LDS row stride of a row-major panel in bytes

// Loads run NB-1 chunks ahead of the math in NB weight register sets, with NB LDS panels.  The
// memory counter retires loads in issue order, so activations and weights of one chunk are
// issued together and at matching distances: waiting for the activations that go to LDS next
// never forces a younger weight load.  Chunk indices past the end are clamped (a few redundant
// loads at the tail keep every chunk one straight-line block, which lets the LDS reads be
// scheduled among the MFMAs).
template <int SPW, int MT, bool GATEUP, bool PACKED, bool XF>
__device__ __forceinline__ void wide_body(const bf16_t* __restrict__ X, const bf16_t* __restrict__ W,
                                          float* __restrict__ out, bf16_t* __restrict__ act, int M, int N, int K,
                                          int tile, int m_base, int c_begin, int c_end, char* lds_raw) {
  constexpr int NB = MT > 8 ? 3 : 4;               // weight register sets and LDS panels
  constexpr int NBX = MT > 8 ? 2 : 4;              // activation register sets
  constexpr int KSTEPS = WKC / 32;
  constexpr int ITEMS = KSTEPS * MT;               // (k step, row tile) pairs of a chunk
  constexpr int BQ = 4;                            // activation fragments read ahead of their MFMAs
  // XF: the activations lie in fragment order.  From 161 rows on beside row-major weights they are row-major (the 256-row
  // body loses 3-5 % with fragments there: gate/up of 512 rows 120 -> 127 us).
  constexpr int UPT = WKC * 2, UNITS = MT * UPT;   // 16-byte units of a row tile's chunk, and of a panel
  constexpr int PASSES = UNITS / 256;
  constexpr int PANEL = XF ? UNITS * 16 : MT * 16 * WXS;
  constexpr int GS = GATEUP ? SPW / 2 : SPW;       // strips per wave and matrix half
  char (*lds)[PANEL] = reinterpret_cast<char (*)[PANEL]>(lds_raw);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // known uniform: addresses split into scalar + lane part
  const int r = lane & 15, kg = lane >> 4;
  const int c_last = c_end - 1;
  // first weight row of strip a of this wave; for gate/up, strips GS.. are the up rows of the same columns
  const int n0 = tile * (64 * GS) + wave * (16 * GS);

  // weights: uniform strip origin + per-lane offset (elements)
  const bf16_t* ws[SPW];
#pragma unroll
  for (int a = 0; a < SPW; ++a) {
    const int row0 = (GATEUP && a >= GS) ? N + n0 + (a - GS) * 16 : n0 + a * 16;
    ws[a] = PACKED ? W + (size_t)(row0 / 16) * (K / 32) * 512 : W + (size_t)row0 * K;
  }
  const unsigned wl = PACKED ? lane * 8 : r * K + kg * 8;
#define SP_WOFF(C, s) (PACKED ? ((size_t)(C) * (WKC / 32) + (s)) * 512 : (size_t)(C)*WKC + (s) * 32)
  // activations: per-thread offset (elements; row tiles or rows past the last one repeat it) + uniform chunk origin
  unsigned xo[PASSES];
  const int xl = XF ? tid * 16 : (tid >> 3) * WXS + (tid & 7) * 16;      // in a panel; passes are XPASS bytes apart
  constexpr int XCHUNK = XF ? WKC * 16 : WKC, XPASS = XF ? 4096 : 32 * WXS;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int u = p * 256 + tid;
    xo[p] = XF ? (unsigned)min((m_base >> 4) + u / UPT, (M - 1) >> 4) * (unsigned)(K * 16) + (u % UPT) * 8
               : (unsigned)min(m_base + (u >> 3), M - 1) * (unsigned)K + (tid & 7) * 8;
  }
  const unsigned bl = XF ? lane * 16 : r * WXS + kg * 16;                // a fragment in its row tile

  u32x4_t wb[NB][SPW][KSTEPS];
  u32x4_t xb[NBX][PASSES];
  f32x4_t acc[SPW][MT];
#pragma unroll
  for (int a = 0; a < SPW; ++a)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[a][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

#define SP_LOAD_X(B, C)                                                                                 \
  {                                                                                                     \
    const bf16_t* xs = X + (size_t)min((C), c_last) * XCHUNK;                                           \
    _Pragma("unroll") for (int p = 0; p < PASSES; ++p)                                                  \
        xb[B][p] = *reinterpret_cast<const u32x4_t*>(xs + xo[p]);                                       \
  }
#define SP_STORE_X(B, BUF)                                                                              \
  _Pragma("unroll") for (int p = 0; p < PASSES; ++p)                                                    \
      *reinterpret_cast<u32x4_t*>(&lds[BUF][p * XPASS + xl]) = xb[B][p];
#define SP_LOAD_W(B, C)                                                                                 \
  {                                                                                                     \
    const int cw = min((C), c_last);                                                                    \
    _Pragma("unroll") for (int a = 0; a < SPW; ++a)                                                     \
        _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s)                                              \
            wb[B][a][s] = *reinterpret_cast<const u32x4_t*>(ws[a] + SP_WOFF(cw, s) + wl);               \
  }
  // item j of a chunk: k step j / MT, row tile j % MT
#define SP_LDS_B(BUF, j)                                                                                \
  (*reinterpret_cast<const bf16x8_t*>(&lds[BUF][XF ? (((j) % MT) * KSTEPS + (j) / MT) * 1024 + bl : ((j) % MT) * 16 * WXS + ((j) / MT) * 64 + bl]))
  // Chunk C, weights in register set B, activations in LDS panel B.  The activations of chunk
  // C+2 go from their register set BX to their panel; that set then takes chunk C+2+NBX and
  // weight set B-1 the weights of chunk C+NB-1.  The last BQ fragment reads already address the
  // next panel, which has been complete since the previous barrier, so the barrier at the end of
  // the chunk is not followed by an exposed LDS round trip.
#define SP_CHUNK(B, BX, C)                                                                              \
  {                                                                                                     \
    const int c_ = (C);                                                                                 \
    SP_STORE_X(BX, ((B) + 2) % NB)                                                                      \
    SP_LOAD_X(BX, c_ + 2 + NBX)                                                                         \
    SP_LOAD_W(((B) + NB - 1) % NB, c_ + NB - 1)                                                         \
    _Pragma("unroll") for (int j = 0; j < ITEMS; ++j) {                                                 \
      const bf16x8_t b = bq[j % BQ];                                                                    \
      if (j + BQ < ITEMS) bq[j % BQ] = SP_LDS_B(B, j + BQ);                                             \
      else bq[j % BQ] = SP_LDS_B(((B) + 1) % NB, j + BQ - ITEMS);                                       \
      _Pragma("unroll") for (int a = 0; a < SPW; ++a) acc[a][j % MT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16( \
          *reinterpret_cast<const bf16x8_t*>(&wb[B][a][j / MT]), b, acc[a][j % MT], 0, 0, 0);           \
    }                                                                                                   \
    /* issue order: panel stores, then per fragment SPW MFMAs, a global load, the next fragment read */ \
    __builtin_amdgcn_sched_group_barrier(0x200, PASSES, 0);                                             \
    _Pragma("unroll") for (int j = 0; j < ITEMS; ++j) {                                                 \
      __builtin_amdgcn_sched_group_barrier(0x008, SPW, 0);                                              \
      if (j < PASSES + SPW * KSTEPS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                 \
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                \
    }                                                                                                   \
    __syncthreads();                                                                                    \
  }

  // prologue: chunks 0 and 1 to their panels, the next NBX activation chunks and the first NB-1
  // weight chunks in flight
#pragma unroll
  for (int i = 0; i < NBX; ++i) SP_LOAD_X(i, c_begin + i)
#pragma unroll
  for (int i = 0; i + 1 < NB; ++i) SP_LOAD_W(i, c_begin + i)
  SP_STORE_X(0, 0)
  SP_STORE_X(1, 1)
  SP_LOAD_X(0, c_begin + NBX)
  SP_LOAD_X(1, c_begin + NBX + 1)
  __syncthreads();
  bf16x8_t bq[BQ];
#pragma unroll
  for (int j = 0; j < BQ; ++j) bq[j] = SP_LDS_B(0, j);
  // unrolled over the common period of the weight and activation set indices
  constexpr int PERIOD = NB == NBX ? NB : NB * NBX;
  for (int c = c_begin; c < c_end; c += PERIOD) {
    SP_CHUNK(0, 2 % NBX, c)
    if (c + 1 < c_end) SP_CHUNK(1 % NB, 3 % NBX, c + 1)
    if (c + 2 < c_end) SP_CHUNK(2 % NB, 4 % NBX, c + 2)
    if (c + 3 < c_end) SP_CHUNK(3 % NB, 5 % NBX, c + 3)
    if (PERIOD > 4) {
      if (c + 4 < c_end) SP_CHUNK(4 % NB, 6 % NBX, c + 4)
      if (c + 5 < c_end) SP_CHUNK(5 % NB, 7 % NBX, c + 5)
    }
  }
#undef SP_CHUNK
#undef SP_LDS_B
#undef SP_LOAD_W
#undef SP_STORE_X
#undef SP_LOAD_X
#undef SP_WOFF

  // lane holds, for activation row m = mt*16 + l%16, output columns (strip base) + 4*(l/16) + 0..3
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = m_base + mt * 16 + r;
    if (m >= M) continue;
    if (GATEUP) {
#pragma unroll
      for (int a = 0; a < GS; ++a) {
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float gte = acc[a][mt][i], up = acc[GS + a][mt][i];
          o[i] = gte / (1.f + __expf(-gte)) * up;
        }
        uint2 pk;
        pk.x = pack_bf16x2(o[0], o[1]);
        pk.y = pack_bf16x2(o[2], o[3]);
        *reinterpret_cast<uint2*>(act + row_at(XF, m, n0 + a * 16 + 4 * kg, N)) = pk;
      }
    } else {
#pragma unroll
      for (int a = 0; a < SPW; ++a)
        *reinterpret_cast<f32x4_t*>(out + ((size_t)blockIdx.y * M + m) * N + n0 + a * 16 + 4 * kg) = acc[a][mt];
    }
  }
}

#ifndef SP_WIDE_OCC8
#define SP_WIDE_OCC8 1
#endif
template <int SPW, int MTMAX, bool GATEUP, bool PACKED, bool XF>
__global__ void __launch_bounds__(256, MTMAX > 8 ? 1 : SP_WIDE_OCC8)
k_gemm_wide(const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, float* __restrict__ out,
            bf16_t* __restrict__ act, int M, int N, int K, int n_tiles, int S) {
  extern __shared__ __attribute__((aligned(16))) char lds_raw[];      // activation panels
  constexpr int WROWS = MTMAX * 16;
  const int n_full = M / WROWS;                     // full row blocks of every column tile
  const int tiles8 = (n_tiles + 7) & ~7;
  const int lin = blockIdx.x;
  int tile, mblk;
  if (lin < tiles8 * n_full) {
    const int xcd = lin & 7, j = lin >> 3;
    tile = (j / n_full) * 8 + xcd;
    mblk = j % n_full;
  } else {
    tile = lin - tiles8 * n_full;
    mblk = n_full;
  }
  if (tile >= n_tiles) return;                      // whole workgroup (the grid is padded to a multiple of 8)
  const int m_base = mblk * WROWS;
  const int chunks_total = K / WKC;
  const int c_begin = (int)(((long long)blockIdx.y * chunks_total) / S);
  const int c_end = (int)(((long long)(blockIdx.y + 1) * chunks_total) / S);
  if (c_begin >= c_end) return;                     // whole workgroup (S never exceeds the chunk count)
  const int rows = M - m_base;                      // uniform over the workgroup
  if (MTMAX > 12 && rows > 192) wide_body<SPW, MTMAX, GATEUP, PACKED, XF>(X, W, out, act, M, N, K, tile, m_base, c_begin, c_end, lds_raw);
  else if (MTMAX > 8 && rows > 128) wide_body<SPW, 12, GATEUP, PACKED, XF>(X, W, out, act, M, N, K, tile, m_base, c_begin, c_end, lds_raw);
  else if (rows > 64) wide_body<SPW, 8, GATEUP, PACKED, XF>(X, W, out, act, M, N, K, tile, m_base, c_begin, c_end, lds_raw);
  else wide_body<SPW, 4, GATEUP, PACKED, XF>(X, W, out, act, M, N, K, tile, m_base, c_begin, c_end, lds_raw);
}

// Launch with the activation panels as dynamic LDS: one array for bodies of every height, with no barrier between them.
template <int SPW, int MT, bool GATEUP, bool PACKED, bool XF>
static hipError_t launch_wide(dim3 grid, hipStream_t st, const bf16_t* X, const bf16_t* W, float* out, bf16_t* act,
                              int M, int N, int K, int n_tiles, int S) {
  constexpr int LDS_BYTES = (MT > 8 ? 3 : 4) * MT * 16 * (XF ? WKC * 2 : WXS);    // NB panels of the tallest body
  static bool ready = false;
  if (!ready) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_wide<SPW, MT, GATEUP, PACKED, XF>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (e != hipSuccess) return e;
    ready = true;
  }
  hipLaunchKernelGGL((k_gemm_wide<SPW, MT, GATEUP, PACKED, XF>), grid, dim3(256), LDS_BYTES, st, X, W, out, act, M, N, K,
                     n_tiles, S);
  return hipGetLastError();
}

// ---- fragment-order weights, many rows ------------------------------------------------------------------------------
// Four waves side by side over 256 weight rows (gate/up: 128 columns, gate and up rows) and RT tiles of 32 activation rows.
// v_mfma_f32_32x32x16_bf16 issues back to back from one wave per SIMD, which the 16 x 16 shape does not (57 % of its rate),
// and gives the same sums; the panels come in by direct-to-LDS loads three chunks of 32 k ahead, as do the weights in
// registers.  Up to RT = 5 two workgroups share a CU.  What sets the time of the products is how many rounds of workgroups
// a shape makes, so the height is chosen by that (wide_plan).  Launches of the 8B shape in 128- and 256-row blocks of the kernel
// above / here, us with the events around them: gate/up 320 rows 110 / 85, 448 rows 107 / 104, 512 rows 112.7 / 114.8, 640 rows
// 163 / 132, 1024 rows 203 / 214; QKV, O and down of 640 rows 48.3 / 40.7, 36.2 / 31.0 and 88.3 / 76.9.  Two layers, 640 rows
// 789 / 679, 1024 rows 1023 / 1023.
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

template <int RT, bool GATEUP>
__global__ void __launch_bounds__(256, RT <= 5 ? 2 : 1)
k_gemm_wide32(const bf16_t* X, const bf16_t* W, float* out, bf16_t* act, int M, int N, int K, int n_tiles, int m_blocks, int S) {
  constexpr int NB = 4, D = 3;                      // panels and weight sets, chunks ahead
  constexpr int BQ = RT == 5 || RT == 7 ? RT : RT == 3 || RT == 6 ? 3 : 4;    // activation fragments read ahead of their MFMAs
  constexpr int BLOCKS = RT * 2, NX = (BLOCKS + 3) / 4, NW = 4;     // fragment blocks of a panel, loads per wave and chunk
  constexpr int PANEL = BLOCKS * 1024;
  constexpr int ITEMS = 2 * RT;                     // (16 k, row tile) pairs of a chunk
  static_assert(ITEMS % BQ == 0, "the fragment queue keeps its place from chunk to chunk");
  // arrays of their own, so that the compiler knows which loads a read has to wait for
  __shared__ __attribute__((aligned(16))) char p0[PANEL];
  __shared__ __attribute__((aligned(16))) char p1[PANEL];
  __shared__ __attribute__((aligned(16))) char p2[PANEL];
  __shared__ __attribute__((aligned(16))) char p3[PANEL];
#define SP_PAN(i) ((i) == 0 ? p0 : (i) == 1 ? p1 : (i) == 2 ? p2 : p3)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, hf = lane >> 5;
  // the row blocks of a column tile get ids that are equal modulo 8: the same XCD, whose L2 holds the tile's weights
  const int lin = blockIdx.x, j8 = lin >> 3;
  const int tile = (j8 / m_blocks) * 8 + (lin & 7), mblk = j8 % m_blocks;
  if (tile >= n_tiles) return;                      // whole workgroup (the grid is padded to a multiple of 8)
  const int chunks = K / 32;
  const int c_begin = (int)(((long long)blockIdx.y * chunks) / S);
  const int c_end = (int)(((long long)(blockIdx.y + 1) * chunks) / S);
  // the wave's two tiles of 32 weight rows: consecutive, or (gate/up) gate rows and the up rows of the same columns
  const int col0 = tile * (GATEUP ? 128 : 256) + wave * (GATEUP ? 32 : 64);
  const bf16_t* w[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) w[a] = W + (size_t)((GATEUP ? a * N + col0 : col0 + a * 32) >> 4) * (K / 32) * 512;
  // lane (r, hf) of an operand: row r, k = 16 * kk + 8 * hf .. + 7
  const int wl = (r >> 4) * (K * 32) + hf * 256 + (r & 15) * 16;
  const int ll = (r >> 4) * 1024 + hf * 256 + (r & 15) * 16;
  const int t0 = mblk * RT * 2, t_last = (M - 1) >> 4;
  // The descriptor starts at the workgroup's row block: the activations of a call may be longer than its 2 GB (16384 rows of
  // d_ff above 65536), a block's offsets stay below 512 * K bytes.
  const bf16_t* xblk = X + (size_t)t0 * (K / 32) * 512;
  int xo[NX], xl[NX];                               // (row tiles and blocks past the last one repeat it)
#pragma unroll
  for (int j = 0; j < NX; ++j) {
    const int b = min(wave * NX + j, BLOCKS - 1);
    xl[j] = b * 1024;
    xo[j] = min(b, t_last - t0) * (K * 32);
  }
  const int lane16 = lane * 16;
  u32x4_t wb[NB][2][2];
  f32x16_t acc[2][RT];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][t][i] = 0.f;
  // The waits count on the order of the loads, a chunk's panel before its weights.  (X and W are not __restrict__: loads of
  // what the compiler takes for constant would be moved past waits and barriers.)
#define SP_LOADS(I, C)                                                                                  \
  {                                                                                                     \
    const bool on_ = (C) < c_end;                                                                       \
    const auto xb_ = buffer_at(xblk, on_);                                                                 \
    _Pragma("unroll") for (int j = 0; j < NX; ++j) load_to_lds(xb_, SP_PAN(I) + xl[j], lane16, (C) * 1024 + xo[j]); \
    __builtin_amdgcn_sched_barrier(0);                                                                  \
    _Pragma("unroll") for (int a = 0; a < 2; ++a) {                                                     \
      const auto wr_ = buffer_at(w[a], on_);                                                            \
      _Pragma("unroll") for (int kk = 0; kk < 2; ++kk)                                                  \
        wb[I][a][kk] = __builtin_amdgcn_raw_buffer_load_b128(wr_, wl, (C) * 1024 + kk * 512, 0);        \
    }                                                                                                   \
  }
#define SP_LDS_B(I, j) (*reinterpret_cast<const bf16x8_t*>(SP_PAN(I) + ((j) % RT) * 2048 + ((j) / RT) * 512 + ll))
  // Chunk C out of panel and weight set I.  What may still be on its way behind the wait: the weights of C + 1 and all loads
  // of C + 2.  Behind the barrier panels C and C + 1 are complete (the last BQ fragment reads
  // already address the next panel) and nobody reads panel C - 1 any more, whose place the loads of chunk C + 3 take.
#define SP_CHUNK(I, C)                                                                                  \
  {                                                                                                     \
    SP_WAIT_VMEM(NX + 2 * NW);                                                                          \
    bare_barrier();                                                                                     \
    SP_LOADS((I + D) % NB, (C) + D)                                                                     \
    __builtin_amdgcn_sched_barrier(0);                                                                  \
    _Pragma("unroll") for (int j = 0; j < ITEMS; ++j) {                                                 \
      const bf16x8_t b = bq[j % BQ];                                                                    \
      if (j + BQ < ITEMS) bq[j % BQ] = SP_LDS_B(I, j + BQ); else bq[j % BQ] = SP_LDS_B((I + 1) % NB, j + BQ - ITEMS); \
      _Pragma("unroll") for (int a = 0; a < 2; ++a) acc[a][j % RT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16( \
          *reinterpret_cast<const bf16x8_t*>(&wb[I][a][j / RT]), b, acc[a][j % RT], 0, 0, 0);           \
    }                                                                                                   \
    _Pragma("unroll") for (int j = 0; j < ITEMS; ++j) {                                                 \
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);                                                \
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                \
    }                                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                  \
  }
#pragma unroll
  for (int i = 0; i < D; ++i) { SP_LOADS(i, c_begin + i) __builtin_amdgcn_sched_barrier(0); }
  SP_WAIT_VMEM(2 * (NX + NW) + NW);
  bare_barrier();
  bf16x8_t bq[BQ];
#pragma unroll
  for (int j = 0; j < BQ; ++j) bq[j] = SP_LDS_B(0, j);
  for (int c = c_begin; c < c_end; c += 4) {
    SP_CHUNK(0, c)
    if (c + 1 < c_end) SP_CHUNK(1, c + 1)
    if (c + 2 < c_end) SP_CHUNK(2, c + 2)
    if (c + 3 < c_end) SP_CHUNK(3, c + 3)
  }
#undef SP_CHUNK
#undef SP_LDS_B
#undef SP_LOADS
  SP_WAIT_VMEM(0);

  // lane (r, hf) holds, for row t * 32 + r, columns 8 * g + 4 * hf + 0..3 of each tile of 32 (g = 0..3)
  if (GATEUP) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int m = t0 * 16 + t * 32 + r;
      if (m >= M) continue;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float gte = acc[0][t][g * 4 + i], up = acc[1][t][g * 4 + i];
          o[i] = gte / (1.f + __expf(-gte)) * up;
        }
        uint2 pk;
        pk.x = pack_bf16x2(o[0], o[1]);
        pk.y = pack_bf16x2(o[2], o[3]);
        *reinterpret_cast<uint2*>(act + frag_at(m, col0 + g * 8 + 4 * hf, N)) = pk;
      }
    }
    return;
  }
  // Partial sums leave as 256 bytes of a row each, put together in a panel per wave (16-byte units of a row exchanged by
  // its number against bank conflicts).
  __syncthreads();
  static_assert(GATEUP || PANEL >= 32 * 256, "32 rows of a wave's 64 columns fit a panel");
  char* buf = SP_PAN(wave);
#pragma unroll
  for (int t = 0; t < RT; ++t) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4_t v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[a][t][g * 4 + i];
        *reinterpret_cast<f32x4_t*>(buf + r * 256 + ((a * 8 + g * 2 + hf) ^ (r & 15)) * 16) = v;
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = i * 4 + (lane >> 4), m = t0 * 16 + t * 32 + row;
      const f32x4_t v = *reinterpret_cast<const f32x4_t*>(buf + row * 256 + ((lane & 15) ^ (row & 15)) * 16);
      if (m < M) *reinterpret_cast<f32x4_t*>(out + ((size_t)blockIdx.y * M + m) * N + col0 + (lane & 15) * 4) = v;
    }
    __builtin_amdgcn_wave_barrier();
  }
#undef SP_PAN
}

// Height of the row blocks and number of k slices.  A column tile's workgroups run on one XCD (ids equal modulo 8), so what
// counts is the XCD with the most tiles: 20 tiles put three on four of them and two on the others (5120 columns, 768 rows: O
// 79.7 us planned over all CUs, 53.3 here).  one, two: us that one workgroup alone on a CU, or two of up to 160 rows side by
// side, take over 4096 k, the least-squares fit of 2090 launches (all heights and slices, 257 to 1024 rows, 2048 to 8192
// columns; residual 4 %; the plan costs 0.4 % of the best choice on average).  A slice costs its partial sums, M * N floats
// written here at 4.6 TB/s and read by the kernel that folds them at 3.4.  gate/up (row_bytes 0): a further round of one
// workgroup a CU costs some 20 us beside its products (700 and 768 rows, heights 6 or 8 / 4: 8B shape 169 / 161, 70B shape 628
// / 602; 70B shape, 512 rows, two rounds of height 8 / 4: 420 / 440).
struct WidePlan { int RT, S; };
static WidePlan wide_plan(int M, int n_tiles, int K, size_t row_bytes, int n_cu, int max_s) {
  static const float one[9] = {0, 0, 0, 0, 60, 68, 77, 87, 96}, two[6] = {0, 0, 0, 0, 103, 117};
  const int xcd_tiles = (n_tiles + 7) / 8, xcd_cus = (n_cu + 7) / 8;
  WidePlan best = {8, 1};
  float best_us = 0.f;
  for (int RT = 4; RT <= 8; ++RT)
    for (int S = 1; S <= max_s; ++S) {
      const int wgs = xcd_tiles * ((M + RT * 32 - 1) / (RT * 32)) * S, n = (wgs + xcd_cus - 1) / xcd_cus;
      const float loop = RT <= 5 ? (n / 2) * two[RT] + (n % 2) * one[RT] : n * one[RT];
      const float more = row_bytes == 0 && RT > 5 ? 22.f * (float)(n - 1) : 0.f;
      const float us = loop * (float)K / (4096.f * (float)S) + more + (float)S * (float)M * (float)row_bytes / 1.95e6f;
      if (best_us == 0.f || us < best_us) { best_us = us; best = {RT, S}; }
    }
  return best;
}
template <bool GATEUP>
static hipError_t launch_wide32(const WidePlan& p, hipStream_t st, const bf16_t* X, const bf16_t* W, float* out, bf16_t* act, int M,
                                int N, int K, int n_tiles) {
  const int m_blocks = (M + p.RT * 32 - 1) / (p.RT * 32);
  const dim3 grid((n_tiles + 7) / 8 * 8 * m_blocks, p.S);
#define SP_GO(RTV) hipLaunchKernelGGL((k_gemm_wide32<RTV, GATEUP>), grid, dim3(256), 0, st, X, W, out, act, M, N, K, n_tiles, m_blocks, p.S)
  switch (p.RT) {
    case 4: SP_GO(4); break;
    case 5: SP_GO(5); break;
    case 6: SP_GO(6); break;
    case 7: SP_GO(7); break;
    default: SP_GO(8); break;
  }
#undef SP_GO
  return hipGetLastError();
}
// From how many rows: gate/up 256 rows 72.0 above / 81.2 us here, 288 rows 105.9 / 86.8; but up to 320 rows where either
// kernel makes one round of workgroups (no XCD has more tiles in three row blocks than CUs), as the one above runs its third
// block at half height (8192 columns, 257 / 320 rows, four layers 3072 wide 696 / 764 above, 713 / 769 us here).  Plain products
// in blocks of 128 rows are level or better up to 384 rows (320 rows: QKV 30.0 / 30.0, O 21.4 / 24.7, down 50.2 / 50.9).
static bool wide32_takes(int M, bool packed, bool gateup, int n_tiles, int n_cu) {
  if (!packed || M <= (gateup ? 256 : 384)) return false;
  return !gateup || M > 320 || (n_tiles + 7) / 8 * 3 > n_cu / 8;
}

// rows per workgroup: 256 once there are enough rows to fill them, else 128
#ifndef SP_WIDE_ROWS
#define SP_WIDE_ROWS(M) ((M) > 384 ? 256 : 128)
#endif
static inline int wide_rows(int M) { return SP_WIDE_ROWS(M); }

hipError_t sp_launch_gemm_wide(const bf16_t* X, bool frag, const bf16_t* W, bool packed, float* out, int M, int N, int K,
                               int n_cu, size_t part_capacity_floats, int* S_out, hipStream_t st) {
  constexpr int SPW = 4;
  if (M < 1 || N % (64 * SPW) || K % WKC || packed != frag) return hipErrorInvalidValue;
  if (wide32_takes(M, packed, false, N / 256, n_cu)) {
    int max_s = K / 32 < 8 ? K / 32 : 8;
    while (max_s > 1 && (size_t)max_s * M * N > part_capacity_floats) --max_s;
    if ((size_t)max_s * M * N > part_capacity_floats) return hipErrorInvalidValue;
    const WidePlan p = wide_plan(M, N / 256, K, (size_t)N * 4, n_cu, max_s);
    *S_out = p.S;
    return launch_wide32<false>(p, st, X, W, out, nullptr, M, N, K, N / 256);
  }
  const int WROWS = wide_rows(M);
  const int n_tiles = N / (64 * SPW), m_blocks = (M + WROWS - 1) / WROWS;
  const int chunks = K / WKC;
  int S = n_cu / (n_tiles * m_blocks);              // split K until about every CU has a workgroup
  if (S < 1) S = 1;
  if (S > 8) S = 8;
  if (S > chunks) S = chunks;
  while (S > 1 && (size_t)S * M * N > part_capacity_floats) --S;
  if ((size_t)S * M * N > part_capacity_floats) return hipErrorInvalidValue;
  *S_out = S;
  const int tiles8 = (n_tiles + 7) / 8 * 8;
  const dim3 grid(tiles8 * m_blocks, S);
  if (packed) return launch_wide<SPW, 8, false, true, true>(grid, st, X, W, out, nullptr, M, N, K, n_tiles, S);
  if (WROWS == 256) return launch_wide<SPW, 16, false, false, false>(grid, st, X, W, out, nullptr, M, N, K, n_tiles, S);
  return launch_wide<SPW, 8, false, false, false>(grid, st, X, W, out, nullptr, M, N, K, n_tiles, S);
}

hipError_t sp_launch_gemm_wide_gateup(const bf16_t* X, bool frag, const bf16_t* W, bool packed, bf16_t* act, int M, int F, int K,
                                      int n_cu, hipStream_t st) {
  constexpr int SPW = 4;                            // two gate strips and two up strips per wave
  constexpr int TW = 64 * (SPW / 2);                // activation columns per workgroup
  if (M < 1 || F % TW || K % WKC || (packed ? !frag : frag && M > 256)) return hipErrorInvalidValue;
  if (wide32_takes(M, packed, true, F / TW, n_cu))
    return launch_wide32<true>(wide_plan(M, F / TW, K, 0, n_cu, 1), st, X, W, nullptr, act, M, F, K, F / TW);
  const int WROWS = wide_rows(M);
  const int n_tiles = F / TW, m_blocks = (M + WROWS - 1) / WROWS;
  const int tiles8 = (n_tiles + 7) / 8 * 8;
  const dim3 grid(tiles8 * m_blocks, 1);
  if (packed) return launch_wide<SPW, 8, true, true, true>(grid, st, X, W, nullptr, act, M, F, K, n_tiles, 1);
  if (frag) return launch_wide<SPW, 8, true, false, true>(grid, st, X, W, nullptr, act, M, F, K, n_tiles, 1);
  if (WROWS == 256) return launch_wide<SPW, 16, true, false, false>(grid, st, X, W, nullptr, act, M, F, K, n_tiles, 1);
  return launch_wide<SPW, 8, true, false, false>(grid, st, X, W, nullptr, act, M, F, K, n_tiles, 1);
}
