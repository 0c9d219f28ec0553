// bf16 projections for 49-160 rows: still a weight stream (one pass over the weights, the activation panel staged
// through LDS once per workgroup), but with this many rows the fragments read back from LDS, not HBM, set the pace if a
// fragment feeds a single MFMA: eight waves with one strip of 16 weight rows each ask LDS for 8 * MT KB per 32 k, at 128
// rows twice the time of the MFMAs they feed.  Here a wave holds two strips and half of the k steps of a chunk, so that
// a fragment feeds two MFMAs, and the two waves that share their strips are folded through LDS at the end (four strips
// per wave measured the same at 128 rows, and at 160 rows the registers do not suffice).  The loop runs without guards
// around its loads up to the last chunks, so that a period of six chunks is one basic block and its waits count exactly.
//
// A workgroup is eight waves over eight strips (plain: 128 columns; gate/up: the CU's even share of the columns as four
// gate strips and the four up strips behind them, the last one short) or six waves over 96 columns, one workgroup per
// CU.  Measured on one 8B layer (forward of the whole layer, before / now): 65 rows 151 -> 134 us, 96 rows 156 -> 141 us,
// 128 rows 171 -> 162 us, 145 rows 190 -> 169 us; 70B layer at 128 rows 399 -> 388 us.
//
//   out[y][m][n] = sum_{k in slice y} X[m][k] * W[n][k]        (f32 partial sums)
//   gate/up:      act[m][f] = silu(X Wg^T) * (X Wu^T)
#include "sp_launch.h"

#define MID_KC 128                       // k per staged chunk
#define MID_XS (MID_KC * 2 + 16)         // LDS row stride of a panel in bytes (conflict-free 16-byte reads)

template <int MT, int NSTRIPS, bool GATEUP, bool PACKED, bool WNT>
__global__ void __launch_bounds__(64 * NSTRIPS)
k_gemm_mid(const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, float* __restrict__ out,
           bf16_t* __restrict__ act, int M, int N, int K, int S, int cpw) {
  constexpr int NS = 2;                   // strips per wave; as many waves share them and split the k steps
  constexpr int NTH = 64 * NSTRIPS;
  constexpr int CW = NSTRIPS / NS;        // waves side by side
  constexpr int KSTEPS = 4 / NS;          // of the chunk's four
  constexpr int ROWS = MT * 16;
  constexpr int UPR = MID_KC / 8, RPP = NTH / UPR, PASSES = (ROWS + RPP - 1) / RPP;
  constexpr bool RAGGED = ROWS % RPP != 0;              // the last staging pass covers fewer rows
  constexpr int PF = 2;                   // weight chunks in flight ahead of the math (three: 1-3 % slower)
  constexpr int NB = PF + 1;              // weight register buffers
  __shared__ __attribute__((aligned(16))) char lds[2][ROWS * MID_XS];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cw = wave % CW, kq = wave / CW;
  const int r = lane & 15, kg = lane >> 4;
  const int chunks = K / MID_KC;
  const int c_begin = (int)(((long long)blockIdx.y * chunks) / S);
  const int c_end = (int)(((long long)(blockIdx.y + 1) * chunks) / S);

  // strip a of this wave: plain, strip cw * NS + a; gate/up, the first half of a wave's strips are gate strips and the
  // second half the up strips of the same columns
  constexpr int GS = GATEUP ? NS / 2 : NS;
  const int col0 = GATEUP ? blockIdx.x * cpw + cw * GS * 16 : blockIdx.x * (16 * NSTRIPS) + cw * NS * 16;
  // addresses as a uniform base per strip and a 32-bit offset per lane (elements), which up and gate strip share
  const bf16_t* w[NS];
  unsigned wl[GS];
#pragma unroll
  for (int a = 0; a < NS; ++a) {
    const int row0 = (GATEUP && a >= GS ? N : 0) + col0 + (a % GS) * 16;
    w[a] = PACKED ? W + ((size_t)(row0 >> 4) * (K / 32) + kq * KSTEPS) * 512 : W + (size_t)row0 * K + kq * (KSTEPS * 32);
  }
#pragma unroll
  for (int g = 0; g < GS; ++g) {
    // a short last group re-reads its last row; its surplus products are dropped at the end
    const int rr = GATEUP ? min(r, cpw - (cw * GS + g) * 16 - 1) : r;
    const int in = (col0 & 15) + rr;      // row inside the strip's first fragment block, or in the one after it
    wl[g] = PACKED ? (unsigned)((in >> 4) * (K / 32) * 512 + (kg * 16 + (in & 15)) * 8) : (unsigned)(rr * K + kg * 8);
  }
  const int xu = tid % UPR, xr = tid / UPR;
  unsigned xo[PASSES];                    // rows past M repeat the last row and multiply into rows that are never stored
#pragma unroll
  for (int p = 0; p < PASSES; ++p) xo[p] = (unsigned)(min(p * RPP + xr, M - 1) * K + xu * 8);

  u32x4_t wb[NB][NS][KSTEPS];
  u32x4_t xb[PASSES];
  f32x4_t acc[NS][MT];
#pragma unroll
  for (int a = 0; a < NS; ++a)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[a][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

  const int c_n = c_end - c_begin;
  // Staggered starting chunks where the rows that the workgroups stream lie a multiple of 8 KB apart and would be at the
  // same offset of it at the same moment: gate/up over row-major weights (8B shape 64 rows 58.8 -> 54.3 us, 145 rows 75.6
  // -> 69.0; nothing gained in fragment order, whose strips are contiguous) and plain products 8192 deep (8192 x 8192, 65
  // rows: 36.3 -> 33.2 us, row-major 40.7 -> 35.5; with K = 4096 slices are four to eight chunks long and lose 1 %, with
  // 14336 and more nothing changes).
  const bool stagger = GATEUP ? !PACKED : K > 4096 && K <= 8192;
  const int rot = stagger && c_n > 1 ? (int)((blockIdx.x >> 3) % (unsigned)c_n) : 0;
#define SP_PC(C) ((GATEUP && PACKED) || (C) + rot < c_end ? (C) + rot : (C) + rot - c_n)
#define SP_LOAD_X(C)                                                                                    \
  _Pragma("unroll") for (int p = 0; p < PASSES; ++p)                                                    \
      xb[p] = *reinterpret_cast<const u32x4_t*>(X + (size_t)SP_PC(C)*MID_KC + xo[p]);
#define SP_STORE_X(BUF)                                                                                 \
  _Pragma("unroll") for (int p = 0; p < PASSES; ++p)                                                    \
      if (!RAGGED || p * RPP + xr < ROWS)                                                               \
        *reinterpret_cast<u32x4_t*>(&lds[BUF][(p * RPP + xr) * MID_XS + xu * 16]) = xb[p];
#define SP_LOAD_W(B, C)                                                                                 \
  _Pragma("unroll") for (int a = 0; a < NS; ++a) _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s) {   \
    const u32x4_t* p_ = reinterpret_cast<const u32x4_t*>(                                               \
        w[a] + (PACKED ? ((size_t)SP_PC(C)*4 + s) * 512 : (size_t)SP_PC(C)*MID_KC + s * 32) + wl[a % GS]);        \
    wb[B][a][s] = WNT ? __builtin_nontemporal_load(p_) : *p_;                                           \
  }
  // Chunk C, weights in register set I % NB, activations in panel I & 1: the next panel goes from registers to LDS,
  // the loads of panel C+2 and of weight chunk C+PF are issued, and the chunk is multiplied.  G: guarded (last chunks).
#define SP_CHUNK(I, C, G)                                                                               \
  {                                                                                                     \
    const int c_ = (C);                                                                                 \
    if (!(G) || c_ + 1 < c_end) { SP_STORE_X(((I) & 1) ^ 1) }                                           \
    if (!(G) || c_ + 2 < c_end) { SP_LOAD_X(c_ + 2) }                                                   \
    if (!(G) || c_ + PF < c_end) { SP_LOAD_W(((I) + PF) % NB, c_ + PF) }                                \
    _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s) _Pragma("unroll") for (int mt = 0; mt < MT; ++mt) { \
      const bf16x8_t b = *reinterpret_cast<const bf16x8_t*>(                                            \
          &lds[(I) & 1][(mt * 16 + r) * MID_XS + ((kq * KSTEPS + s) * 32 + kg * 8) * 2]);               \
      _Pragma("unroll") for (int a = 0; a < NS; ++a) acc[a][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16( \
          *reinterpret_cast<const bf16x8_t*>(&wb[(I) % NB][a][s]), b, acc[a][mt], 0, 0, 0);             \
    }                                                                                                   \
    __syncthreads();                                                                                    \
  }
  if (c_begin < c_end) {
    SP_LOAD_X(c_begin)
    SP_LOAD_W(0, c_begin)
    if (c_begin + 1 < c_end) { SP_LOAD_W(1, c_begin + 1) }
    SP_STORE_X(0)
    if (c_begin + 1 < c_end) { SP_LOAD_X(c_begin + 1) }
  }
  __syncthreads();
  constexpr int PERIOD = 2 * NB;          // chunk index modulo this fixes every buffer
  static_assert(PF == 2 && PERIOD == 6, "the loops below are written for two chunks ahead");
  int c = c_begin;
  for (; c + PERIOD - 1 + PF < c_end; c += PERIOD) {
    SP_CHUNK(0, c, false)
    SP_CHUNK(1, c + 1, false)
    SP_CHUNK(2, c + 2, false)
    SP_CHUNK(3, c + 3, false)
    SP_CHUNK(4, c + 4, false)
    SP_CHUNK(5, c + 5, false)
  }
  for (; c < c_end; c += PERIOD) {
    SP_CHUNK(0, c, true)
    if (c + 1 < c_end) SP_CHUNK(1, c + 1, true)
    if (c + 2 < c_end) SP_CHUNK(2, c + 2, true)
    if (c + 3 < c_end) SP_CHUNK(3, c + 3, true)
    if (c + 4 < c_end) SP_CHUNK(4, c + 4, true)
    if (c + 5 < c_end) SP_CHUNK(5, c + 5, true)
  }
#undef SP_CHUNK
#undef SP_PC
#undef SP_LOAD_W
#undef SP_STORE_X
#undef SP_LOAD_X

  // Fold the NS waves that share their strips: strip by strip, every wave leaves the row tiles that are not its own
  // (tile mt belongs to wave mt % NS of the sharers) and adds the other waves' products of its own tiles, in order.
  f32x4_t* fold = reinterpret_cast<f32x4_t*>(&lds[0][0]);           // [waves][MT][64 lanes]
  static_assert(NSTRIPS * MT * 64 * 16 <= (int)sizeof(lds), "one strip of every wave fits the panels");
#pragma unroll
  for (int a = 0; a < NS; ++a) {
    if (a > 0) __syncthreads();           // (the last chunk ended with a barrier)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (mt % NS != kq) fold[(wave * MT + mt) * 64 + lane] = acc[a][mt];
    __syncthreads();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if (mt % NS != kq) continue;
      f32x4_t t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < NS; ++q) t += q == kq ? acc[a][mt] : fold[((q * CW + cw) * MT + mt) * 64 + lane];
      acc[a][mt] = t;
    }
  }

  // lane holds, for row m = mt*16 + l%16 of its own tiles, columns (strip base) + 4*(l/16) + 0..3
  if (GATEUP) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = mt * 16 + r;
      if (mt % NS != kq || m >= M) continue;
#pragma unroll
      for (int g = 0; g < GS; ++g) {
        if (4 * kg >= cpw - (cw * GS + g) * 16) continue;           // columns past a short last group
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float gte = acc[g][mt][i], up = acc[GS + g < NS ? GS + g : 0][mt][i];
          o[i] = gte / (1.f + __expf(-gte)) * up;
        }
        uint2 pk;
        pk.x = pack_bf16x2(o[0], o[1]);
        pk.y = pack_bf16x2(o[2], o[3]);
        *reinterpret_cast<uint2*>(act + (size_t)m * N + col0 + g * 16 + 4 * kg) = pk;
      }
    }
    return;
  }
  // Partial sums leave in whole rows of the workgroup's columns, put together in LDS: a store instruction then writes
  // 1 KB of consecutive addresses instead of 64 bytes in each of 16 rows.
  constexpr int WCOLS = 16 * NSTRIPS, LSF = WCOLS + 4;    // columns, and floats per LDS row
  static_assert(ROWS * LSF * 4 <= (int)sizeof(lds), "the row tile fits the panels' LDS");
  float* tile = reinterpret_cast<float*>(&lds[0][0]);
  __syncthreads();
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
    if (mt % NS == kq) {
#pragma unroll
      for (int a = 0; a < NS; ++a)
        *reinterpret_cast<f32x4_t*>(tile + (mt * 16 + r) * LSF + (cw * NS + a) * 16 + 4 * kg) = acc[a][mt];
    }
  __syncthreads();
  constexpr int UPW = WCOLS / 4;                          // 16-byte units per row
  for (int idx = tid; idx < ROWS * UPW; idx += NTH) {
    const int row = idx / UPW, u = idx - row * UPW;
    if (row < M)
      *reinterpret_cast<f32x4_t*>(out + ((size_t)blockIdx.y * M + row) * N + blockIdx.x * WCOLS + u * 4) =
          *reinterpret_cast<const f32x4_t*>(tile + row * LSF + u * 4);
  }
}

// row tiles of a launch: the kernel is compiled for these heights
static inline int mid_tiles(int M) { return M <= 64 ? 4 : M <= 96 ? 6 : M <= 128 ? 8 : 10; }
#define SP_BY_TILES(GO)                  \
  switch (mid_tiles(M)) {                \
    case 4: GO(4); break;                \
    case 6: GO(6); break;                \
    case 8: GO(8); break;                \
    default: GO(10); break;              \
  }

template <int NSTRIPS, bool PACKED, bool WNT>
static hipError_t launch_plain(dim3 grid, hipStream_t st, const bf16_t* X, const bf16_t* W, float* out, int M, int N, int K, int S) {
#define SP_GO(MTV) \
  hipLaunchKernelGGL((k_gemm_mid<MTV, NSTRIPS, false, PACKED, WNT>), grid, dim3(64 * NSTRIPS), 0, st, X, W, out, nullptr, M, N, K, S, 0)
  SP_BY_TILES(SP_GO)
#undef SP_GO
  return hipGetLastError();
}

template <bool PACKED>
static hipError_t launch_gateup(int n_cu, hipStream_t st, const bf16_t* X, const bf16_t* W, bf16_t* act, int M, int F, int K) {
#define SP_GO(MTV) \
  hipLaunchKernelGGL((k_gemm_mid<MTV, 8, true, PACKED, true>), dim3(n_cu), dim3(512), 0, st, X, W, nullptr, act, M, F, K, 1, F / n_cu)
  SP_BY_TILES(SP_GO)
#undef SP_GO
  return hipGetLastError();
}

// How a plain product is cut: columns per workgroup and k slices, one workgroup per CU (every further slice costs M*N*4
// bytes written here and read again by the folding kernel).  96 columns where those tiles divide the CUs evenly and tiles
// of 128 do not (N = 6144 on 256 CUs: 64 tiles x 4 slices of equal length instead of 48 x 5 of 6 or 7 chunks).  Six waves
// on four SIMDs leave half of the matrix cores idle for half of the time, which counts as soon as these, not the
// weights, set the pace: from 97 rows on, only for short slices (one layer, us with 96 / 128 columns: 6144 wide, slices of
// 12 to 32 chunks, 65 rows 198 / 196, 97 rows 228 / 209, 160 rows 259 / 243; 3072 wide, slices of 3 and 8 chunks, 65 rows
// 104 / 106, 97 rows 117 / 117, 160 rows 142 / 146).
struct MidCut { int cols, S; };
static MidCut mid_cut(int M, int N, int K, int n_cu) {
  const int chunks = K / MID_KC;
  const bool even96 = N % 96 == 0 && n_cu % (N / 128) != 0 && n_cu % (N / 96) == 0;
  const bool six = even96 && (M <= 96 || chunks <= 8 * (n_cu / (N / 96)));
  return {six ? 96 : 128, n_cu / (N / (six ? 96 : 128))};
}

// Where this kernel is the faster one (us per launch, k_gemm_bf16 or k_gemm_wide against this one, 8B and 70B shapes):
// gate/up 64 rows 45.5 / 43.7, 128 rows 60.4 / 54.6, 145 rows 70.2 / 59.3, at 48 rows 43.5 / 49.8; down, 14336 or 28672
// deep, 64 rows 28.1 / 26.8 and 83 / 77, 145 rows 42.1 / 35.9; QKV and O of both shapes lose up to 8 % at 64 rows (their
// k slices are four to eight chunks long) and gain from 65 on (145 rows 25.5 / 24.4 and 22.2 / 18.6).  From 161 rows on
// the register-blocked kernel is level, and with twelve row tiles slower here.
// Over other widths (one layer, us, k_gemm_bf16 against this one): up to 64 rows it loses in tiles of 96 columns (6144
// wide, 64 rows 199 / 205) and where the columns leave two slices or one (12288 wide, row-major 534 / 550).  With seven
// and eight row tiles a launch costs 0.8 us more here, the fold of the waves that share their strips, which slices of one
// chunk do not earn back (97 rows: 768 wide 60.5 / 62.9, 1024 wide 69.5 / 71.8; with two chunks in QKV alone, 2048 wide,
// 94.5 / 92.5), nor do two slices of a wide matrix (12288 wide 451 / 470, row-major 605 / 638).  65-96 and 129-160 rows:
// level (768 wide) to 8 % faster throughout.
bool sp_gemm_mid_takes(int M, int N, int K, int n_cu) {
  if (M <= 48 || M > 160 || N % 128 || K % MID_KC) return false;
  const MidCut cut = mid_cut(M, N, K, n_cu);
  if (M <= 64) return K > 8192 && cut.cols == 128 && cut.S >= 3;
  if (M > 96 && M <= 128) return cut.S >= 3 && K / MID_KC >= 2 * (cut.S < 16 ? cut.S : 16);
  return true;
}
bool sp_gemm_mid_takes_gateup(int M, int F, int K, int n_cu) {
  return M > 48 && M <= 160 && K % MID_KC == 0 && n_cu > 0 && F % n_cu == 0 && (F / n_cu) % 8 == 0 && F / n_cu > 48 &&
         F / n_cu <= 64;
}

hipError_t sp_launch_gemm_mid(const bf16_t* X, const bf16_t* W, bool packed, float* out, int M, int N, int K, int n_cu,
                              int max_split, size_t part_capacity_floats, int* S_out, hipStream_t st, bool resident) {
  if (!sp_gemm_mid_takes(M, N, K, n_cu)) return hipErrorInvalidValue;
  const MidCut cut = mid_cut(M, N, K, n_cu);
  const bool six = cut.cols == 96;
  const int tiles = N / cut.cols, chunks = K / MID_KC;
  int S = cut.S;
  if (S > max_split) S = max_split;
  if (S > chunks) S = chunks;
  while (S > 1 && (size_t)S * M * N > part_capacity_floats) --S;
  if (S < 1) S = 1;
  if ((size_t)S * M * N > part_capacity_floats) return hipErrorInvalidValue;
  *S_out = S;
  const dim3 grid(tiles, S);
  if (six && resident) return packed ? launch_plain<6, true, false>(grid, st, X, W, out, M, N, K, S) : launch_plain<6, false, false>(grid, st, X, W, out, M, N, K, S);
  if (six) return packed ? launch_plain<6, true, true>(grid, st, X, W, out, M, N, K, S) : launch_plain<6, false, true>(grid, st, X, W, out, M, N, K, S);
  if (resident) return packed ? launch_plain<8, true, false>(grid, st, X, W, out, M, N, K, S) : launch_plain<8, false, false>(grid, st, X, W, out, M, N, K, S);
  return packed ? launch_plain<8, true, true>(grid, st, X, W, out, M, N, K, S) : launch_plain<8, false, true>(grid, st, X, W, out, M, N, K, S);
}

hipError_t sp_launch_gemm_mid_gateup(const bf16_t* X, const bf16_t* W, bool packed, bf16_t* act, int M, int F, int K, int n_cu,
                                     hipStream_t st) {
  if (!sp_gemm_mid_takes_gateup(M, F, K, n_cu)) return hipErrorInvalidValue;
  return packed ? launch_gateup<true>(n_cu, st, X, W, act, M, F, K) : launch_gateup<false>(n_cu, st, X, W, act, M, F, K);
}
