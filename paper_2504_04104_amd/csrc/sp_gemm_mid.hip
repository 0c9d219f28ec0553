// bf16 products of up to 160 rows (gate/up 192): a weight stream, one pass over the weights, with the activation panel
// staged through LDS once per workgroup.  Two things bound it beside HBM.  The fragments read back from LDS, if each feeds a
// single MFMA: eight waves with one strip of 16 weight rows each ask LDS for 8 * MT KB per 32 k, at 128 rows twice the time of
// the MFMAs they feed, so a wave holds two strips and half of the k steps of a chunk and the two waves that share their strips
// are folded through LDS at the end.  And the panel's way from L2 into the CU, which moves 1 KB of consecutive addresses at
// 120 B/ns per CU, 128-byte pieces at 78 and 64-byte pieces at 38: X comes in fragment order.
//
// Panels come in by direct-to-LDS loads of waves of their own.  A wave's loads return in order, so one that waits for its
// piece of the panel would wait for all its older weight loads too; the loading waves need no registers for either.
// Row-major weights take the same way: a wave loads whole 128-byte lines of its rows to LDS (the 16-byte units swizzled over
// the banks) and reads fragments back, 6.3-6.5 TB/s against some 5 for 64-byte pieces in operand layout; so do weights
// in fragment order where the registers are needed for the sums (PlainPipe, GateupPipe).  A period of the ring is one basic
// block without guards around its loads (a load past the end goes through an empty buffer descriptor), so that its waits
// count exactly.
//
// A workgroup covers eight strips (plain: 128 columns; gate/up: the CU's even share of the columns as gate strips and the up
// strips behind them, the last one short), twelve (96 columns: six waves) or, gate/up of 97-112 columns per CU, fourteen, one
// workgroup per CU.  Two 8B or one 70B layer, the kernels before / here, us: 8B row-major 16 rows 262 / 212, 64 rows 287 / 238, 160 rows
// 376 / 320; 70B row-major 17 rows 371 / 301, 64 rows 412 / 320, 128 rows 476 / 372, 160 rows 666 / 405; 70B in fragment order
// 160 rows 562 / 392; 12288 wide in fragment order 112 rows 594 / 555.
//
//   out[y][m][n] = sum_{k in slice y} X[m][k] * W[n][k]        (f32 partial sums)
//   gate/up:      act[m][f] = silu(X Wg^T) * (X Wu^T)
#include <type_traits>

#include "sp_launch.h"

#define MID_NS 2                         // strips of 16 weight rows per wave
#define MID_NPR 2                        // waves that bring the panels in
#define MID_KC 128                       // slices of plain products are cut between blocks of this many k

// MT row tiles; CW waves side by side, KQ that share their strips and cut a chunk's k steps between them; chunks of KC k;
// activation panels D chunks ahead, weights PF chunks ahead; NPR waves that bring the panels in.
template <int MT, int CW, int KQ, bool GATEUP, bool PACKED, bool WNT, int KC, int D, int PF, int NPR, bool WL>
__global__ void __launch_bounds__(64 * (CW * KQ + NPR))
k_gemm_mid(const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, float* __restrict__ out,
           bf16_t* __restrict__ act, int M, int N, int K, int S, int cpw, const float* ssq = nullptr, float eps = 0.f) {
  constexpr int NS = MID_NS;
  constexpr int NMM = CW * KQ, NTH = 64 * (NMM + NPR);  // waves that multiply, threads
  constexpr int CS = KC / 32, KSTEPS = CS / KQ;         // k steps of a chunk, and of a wave in it
  constexpr int ROWS = MT * 16;
  constexpr int BLOCKS = MT * CS, NX = BLOCKS / NPR;    // 1 KB fragment blocks of a panel, and of a loading wave in it
  constexpr int PANEL = BLOCKS * 1024;
  constexpr int NP = D + 1, NB = PF + 1;                // panels, weight register buffers
  constexpr int OT = (MT + KQ - 1) / KQ;                // row tiles a wave finishes
  constexpr int FOLD_BYTES = KQ > 1 ? NMM * OT * 1024 : 0;
  constexpr int WCOLS = 16 * NS * CW, LSF = WCOLS + 4;  // columns, and floats per LDS row of the plain products
  constexpr int OUT_BYTES = GATEUP ? 0 : ROWS * LSF * 4;
  constexpr int END_BYTES = FOLD_BYTES > OUT_BYTES ? FOLD_BYTES : OUT_BYTES;
  // Row-major weights: a wave's rows come in as whole 128-byte lines (64 k), straight to LDS, and are read back as
  // fragments; one array per set, so that the compiler knows which loads a read has to wait for.
  constexpr int WSET = !WL ? 16 : NMM * NS * KSTEPS * 1024;
  static_assert(PACKED || KSTEPS % 2 == 0, "whole lines of row-major weights");
  __shared__ __attribute__((aligned(16))) char wl0[WSET];
  __shared__ __attribute__((aligned(16))) char wl1[WSET];
  __shared__ __attribute__((aligned(16))) char wl2[NB > 2 ? WSET : 16];
#define SP_WSET(B) ((B) == 0 ? wl0 : (B) == 1 ? wl1 : wl2)
  static_assert(!WL || NB <= 3, "weight sets");
  static_assert(BLOCKS % NPR == 0 && CS % KQ == 0 && KQ <= 2 && (D - 1) * NX < 64 && PF >= 1 && PF <= 3, "shape of the pipeline");
  __shared__ __attribute__((aligned(16))) char lds[NP * PANEL > END_BYTES ? NP * PANEL : END_BYTES];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cw = wave % CW, kq = wave / CW;             // (kq == KQ and beyond: loading waves)
  const bool mm = wave < NMM;
  const int r = lane & 15, kg = lane >> 4;
  const int chunks = K / KC;
  const int c_begin = (int)(((long long)blockIdx.y * chunks) / S);
  const int c_end = (int)(((long long)(blockIdx.y + 1) * chunks) / S);
  const int c_n = c_end - c_begin;
  // Staggered starting chunks where the rows or strips that the workgroups stream lie a multiple of 8 KB apart and would be
  // at the same offset of it at the same moment: gate/up over row-major weights (8B shape 64 rows 58.8 -> 54.3 us, 145 rows
  // 75.6 -> 69.0) and, up to 96 rows, over weights in fragment order (8B layers, on several machines with buffers at many places:
  // 33-48 rows level to 1 % faster, 56-64 from 0.8 % slower to 1.4 % faster, mostly faster, 72-96 0.4-1.5 % faster; 70B shape 33-40
  // rows level to 1 % slower, 48-96 0.3-0.5 % faster; with more rows level), and plain products 8192 deep (8192 x 8192, 65 rows:
  // 36.3 -> 33.2 us, row-major 40.7 -> 35.5; with K = 4096 slices are four to eight chunks long and lose 1 %, with 14336 and
  // more nothing changes).
  const bool stagger = GATEUP ? !PACKED || MT <= 6 : K > 4096 && K <= 8192;
  const int rot = stagger && c_n > 1 ? (int)((blockIdx.x >> 3) % (unsigned)c_n) : 0;
#define SP_PC(C) ((GATEUP && PACKED && MT > 6) || (C) + rot < c_end ? (C) + rot : (C) + rot - c_n)

  // strip a of a wave: plain, strip cw * NS + a; gate/up, a gate strip and the up strip of the same columns
  constexpr int GS = GATEUP ? NS / 2 : NS;
  const int col0 = GATEUP ? blockIdx.x * cpw + cw * GS * 16 : blockIdx.x * WCOLS + cw * NS * 16;
  f32x4_t acc[NS][MT];
#pragma unroll
  for (int a = 0; a < NS; ++a)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[a][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

  // one row tile of gate/up: the rows may come without their RMSNorm, whose scale is then a factor of the products
  constexpr bool SCALED = GATEUP && MT == 1;
  __shared__ float s_tot[SCALED ? 16 : 1];
  constexpr int SQW = !SCALED ? 1 : 16 % NMM == 0 ? NMM : 4;      // multiplying waves that share the 16 rows evenly
  static_assert(SQW <= NMM, "the row sums belong to multiplying waves");
  RowSquares<64 * SQW> sq;
  if (SCALED && wave < SQW && ssq) sq.load(ssq, K / 16, M);

  // One barrier per chunk.  Behind that of chunk C, panel C is complete and nobody reads panel C - 1 any more, whose
  // place panel C + D takes.  Loads past the last chunk go to an empty buffer: they cost an issue slot and keep every
  // chunk's wait the same.
  if (!mm) {
    const int pr = wave - NMM;
    // Row tiles past the last one repeat it, and of up to four tiles rows past M the last one, so that half of a nearly empty
    // tile's lines are not asked for (33 rows, two 8B layers 228.8 -> 227.8 us; of eight tiles whole blocks are faster, 108
    // rows 286.0 against 289.3); they multiply into rows that are never stored.
    int xo[NX], xl[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      const int b = pr * NX + j;
      const int tile = min(b / CS, (M - 1) >> 4);
      xo[j] = tile * (K * 32) + (b % CS) * 1024;
      xl[j] = (kg * 16 + (MT <= 4 ? min(r, M - 1 - tile * 16) : r)) * 16;
    }
    int pan = pr * NX * 1024;
    auto load_x = [&](int c) {
      const auto buf = buffer_at(X, c < c_end);
      const int pc = SP_PC(c) * (KC * 32);
#pragma unroll
      for (int j = 0; j < NX; ++j) load_to_lds(buf, lds + pan + j * 1024, xl[j], pc + xo[j]);
      pan += PANEL;
      if (pan >= NP * PANEL) pan -= NP * PANEL;
    };
#pragma unroll
    for (int i = 0; i < D; ++i) load_x(c_begin + i);
    for (int c = c_begin; c < c_end; ++c) {
      SP_WAIT_VMEM((D - 1) * NX);
      bare_barrier();
      load_x(c + D);
    }
    SP_WAIT_VMEM(0);
  } else {
    // addresses as a uniform base per strip and an offset per lane (bytes), which up and gate strip share
    const bf16_t* w[NS];
    int wl[GS][PACKED ? 1 : 2];
#pragma unroll
    for (int a = 0; a < NS; ++a) {
      const int row0 = (GATEUP && a >= GS ? N : 0) + col0 + (a % GS) * 16;
      w[a] = PACKED ? W + ((size_t)(row0 >> 4) * (K / 32) + kq * KSTEPS) * 512 : W + (size_t)row0 * K + kq * (KSTEPS * 32);
    }
#pragma unroll
    for (int g = 0; g < GS; ++g) {
      // a short last group re-reads its last row; its surplus products are dropped at the end
      const int last = GATEUP ? cpw - (cw * GS + g) * 16 - 1 : 15;
      if (PACKED) {
        const int in = (col0 & 15) + min(r, last);   // row inside the strip's first fragment block, or in the one after it
        wl[g][0] = (in >> 4) * (K * 32) + (kg * 16 + (in & 15)) * 16;
      } else {
        // eight rows of 128 bytes per load; within a row the eight 16-byte units are exchanged by the row's number, which
        // spreads a fragment's units over the LDS banks
#pragma unroll
        for (int h = 0; h < 2; ++h) wl[g][PACKED ? 0 : h] = min(h * 8 + (lane >> 3), last) * (K * 2) + ((lane & 7) ^ (lane >> 3)) * 16;
      }
    }
    u32x4_t wb[!WL ? NB : 1][NS][KSTEPS];
    const int wbase = wave * (NS * KSTEPS * 1024), wread = wbase + (PACKED ? lane * 16 : (r >> 3) * 1024 + (r & 7) * 128);
#define SP_LOAD_W(B, C)                                                                                 \
  {                                                                                                     \
    const bool on_ = (C) < c_end;                                                                       \
    const int pc_ = SP_PC(C);                                                                           \
    _Pragma("unroll") for (int a = 0; a < NS; ++a) {                                                    \
      const auto buf_ = buffer_at(w[a], on_);                                                           \
      _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s) {                                              \
        if (!WL)                                                                                        \
          wb[!WL ? (B) : 0][a][s] = __builtin_amdgcn_raw_buffer_load_b128(buf_, wl[a % GS][0], (pc_ * CS + s) * 1024, WNT ? 2 : 0); \
        else if (PACKED)                                                                                \
          load_to_lds<WNT>(buf_, SP_WSET(B) + wbase + (a * KSTEPS + s) * 1024, wl[a % GS][0], (pc_ * CS + s) * 1024); \
        else    /* load s: rows (s % 2) * 8 .. + 7, k group s / 2 */                                    \
          load_to_lds<WNT>(buf_, SP_WSET(B) + wbase + (a * KSTEPS + s) * 1024, wl[a % GS][PACKED ? 0 : s % 2], (pc_ * KC + s / 2 * 64) * 2); \
      }                                                                                                 \
    }                                                                                                   \
    __builtin_amdgcn_sched_barrier(0);                                                                  \
  }
  // row-major: fragments of set B, strip a, k step s, out of LDS
#define SP_READ_W(B)                                                                                    \
  if (WL) {                                                                                             \
    SP_WAIT_VMEM(PF * NS * KSTEPS);       /* the sets behind this one */                                \
    _Pragma("unroll") for (int a = 0; a < NS; ++a) _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s)   \
      wb[0][a][s] = *reinterpret_cast<const u32x4_t*>(SP_WSET(B) + wread + (PACKED ? (a * KSTEPS + s) * 1024 : (a * KSTEPS + s / 2 * 2) * 1024 + ((s % 2 * 4 + kg) ^ (r & 7)) * 16)); \
  }
    int pan = lane * 16;
#define SP_CHUNK(B, C)                                                                                  \
  if ((C) < c_end) {                                                                                    \
    bare_barrier();                                                                                     \
    SP_LOAD_W(((B) + PF) % NB, (C) + PF)                                                                \
    SP_READ_W(B)                                                                                        \
    _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s) _Pragma("unroll") for (int mt = 0; mt < MT; ++mt) { \
      const bf16x8_t b = *reinterpret_cast<const bf16x8_t*>(lds + pan + (mt * CS + kq * KSTEPS + s) * 1024); \
      _Pragma("unroll") for (int a = 0; a < NS; ++a) acc[a][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16( \
          *reinterpret_cast<const bf16x8_t*>(&wb[!WL ? (B) : 0][a][s]), b, acc[a][mt], 0, 0, 0);     \
    }                                                                                                   \
    pan = pan + PANEL >= NP * PANEL ? pan + PANEL - NP * PANEL : pan + PANEL;                           \
    __builtin_amdgcn_sched_barrier(0);                                                                  \
  }
#pragma unroll
    for (int i = 0; i < PF; ++i) SP_LOAD_W(i, c_begin + i)
    for (int c = c_begin; c < c_end; c += NB) {
      SP_CHUNK(0, c)
      SP_CHUNK(1, c + 1)
      if (NB > 2) SP_CHUNK(2 % NB, c + 2)
      if (NB > 3) SP_CHUNK(3 % NB, c + 3)
    }
#undef SP_CHUNK
#undef SP_LOAD_W
#undef SP_READ_W
#undef SP_WSET
  }
#undef SP_PC

  if (SCALED && wave < SQW && ssq) sq.post(ssq, K / 16, M, s_tot);
  if (SCALED && KQ == 1) __syncthreads();       // (with two waves per strip the fold has its barriers)
  if (KQ > 1) {
    // Fold the two waves that share their strips: strip by strip, a wave leaves the row tiles that are not its own (tile
    // mt belongs to wave mt % 2) and adds the other's products of its own tiles, in order.
    f32x4_t* fold = reinterpret_cast<f32x4_t*>(lds);               // [waves][OT][64 lanes]
#pragma unroll
    for (int a = 0; a < NS; ++a) {
      __syncthreads();                    // the panels, or the strip before, are no longer read
      if (mm) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          if (mt % KQ != kq) fold[(wave * OT + mt / KQ) * 64 + lane] = acc[a][mt];
      }
      __syncthreads();
      if (mm) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          if (mt % KQ != kq) continue;
          const f32x4_t o = fold[(((KQ - 1 - kq) * CW + cw) * OT + mt / KQ) * 64 + lane];
          acc[a][mt] = kq == 0 ? acc[a][mt] + o : o + acc[a][mt];
        }
      }
    }
  }

  // lane holds, for row m = mt*16 + l%16 of its own tiles, columns (strip base) + 4*(l/16) + 0..3
  if (GATEUP) {
    if (!mm) return;
    float row_scale = 1.f;
    if (SCALED && ssq) row_scale = rsqrtf(s_tot[min(r, M - 1)] / (float)K + eps);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = mt * 16 + r;
      if (mt % KQ != kq || m >= M) continue;
#pragma unroll
      for (int g = 0; g < GS; ++g) {
        if (4 * kg >= cpw - (cw * GS + g) * 16) continue;           // columns past a short last group
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float gte = SCALED ? acc[g][mt][i] * row_scale : acc[g][mt][i];
          const float up = SCALED ? acc[GS + g < NS ? GS + g : 0][mt][i] * row_scale : acc[GS + g < NS ? GS + g : 0][mt][i];
          o[i] = gte / (1.f + __expf(-gte)) * up;
        }
        uint2 pk;
        pk.x = pack_bf16x2(o[0], o[1]);
        pk.y = pack_bf16x2(o[2], o[3]);
        *reinterpret_cast<uint2*>(act + frag_at(m, col0 + g * 16 + 4 * kg, N)) = pk;
      }
    }
    return;
  }
  // Partial sums leave in whole rows of the workgroup's columns, put together in LDS: a store instruction then writes
  // 1 KB of consecutive addresses instead of 64 bytes in each of 16 rows.
  float* tile = reinterpret_cast<float*>(lds);
  __syncthreads();
  if (mm) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (mt % KQ == kq) {
#pragma unroll
        for (int a = 0; a < NS; ++a)
          *reinterpret_cast<f32x4_t*>(tile + (mt * 16 + r) * LSF + (cw * NS + a) * 16 + 4 * kg) = acc[a][mt];
      }
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
static inline int mid_tiles(int M) { return M <= 64 ? (M + 15) / 16 : M <= 96 ? 6 : M <= 128 ? 8 : M <= 160 ? 10 : 12; }
#define SP_BY_TILES(GO)       \
  switch (mid_tiles(M)) {     \
    case 1: GO(1) break;      \
    case 2: GO(2) break;      \
    case 3: GO(3) break;      \
    case 4: GO(4) break;      \
    case 6: GO(6) break;      \
    case 8: GO(8) break;      \
    case 10: GO(10) break;    \
    default: GO(12) break;    \
  }

// Chunk length, how far panels and weights are ahead, loading waves, and whether the weights go through LDS, within
// 160 KB of LDS and 168 registers.
template <int KC_, int D_, int PF_, bool WL_> struct MidPipe {
  static constexpr int KC = KC_, D = D_, PF = PF_;
  static constexpr bool WL = WL_;
};
template <int MT, bool PACKED, bool SHORT> struct PlainPipe
    : std::conditional_t<!PACKED, std::conditional_t<(MT <= 4), MidPipe<128, 2, 2, true>, std::conditional_t<(MT <= 6), MidPipe<128, 2, 1, true>, MidPipe<128, 1, 1, true>>>,
                         std::conditional_t<(MT > 8 || (MT == 8 && SHORT)), MidPipe<64, 3, 2, true>,
                                            std::conditional_t<(MT <= 6), MidPipe<128, 2, 1, true>, MidPipe<128, 2, 2, false>>>> {};
template <int MT, int KQ, bool PACKED> struct GateupPipe
    : std::conditional_t<KQ == 1, std::conditional_t<(MT <= 8 || !PACKED), MidPipe<64, MT <= 8 ? 3 : 2, MT <= 8 && PACKED ? 2 : 1, true>, MidPipe<128, 2, 1, false>>,
                         std::conditional_t<(MT <= 6), MidPipe<128, 2, MT <= 4 ? 2 : 1, true>,
                                            std::conditional_t<(MT > 10), MidPipe<64, 3, 3, false>,
                                                               std::conditional_t<PACKED, MidPipe<128, 2, 2, false>, MidPipe<128, 1, 1, true>>>>> {};

template <int NSTRIPS, bool PACKED, bool WNT, bool SHORT>
static hipError_t launch_plain(dim3 grid, hipStream_t st, const bf16_t* X, const bf16_t* W, float* out, int M, int N, int K, int S) {
#define SP_GO(MTV)                                                                                                        \
  if constexpr (MTV <= 10) {                                                                                              \
    typedef PlainPipe<MTV, PACKED, SHORT> P;                                                                              \
    hipLaunchKernelGGL((k_gemm_mid<MTV, NSTRIPS / 2, 2, false, PACKED, WNT, P::KC, P::D, P::PF, MID_NPR, P::WL>), grid,   \
                       dim3(64 * (NSTRIPS + MID_NPR)), 0, st, X, W, out, nullptr, M, N, K, S, 0, nullptr, 0.f);           \
  } else return hipErrorInvalidValue;
  SP_BY_TILES(SP_GO)
#undef SP_GO
  return hipGetLastError();
}

// gate/up: CW groups of 16 columns
template <int CW, int KQ, bool PACKED>
static hipError_t launch_gateup(int n_cu, hipStream_t st, const bf16_t* X, const bf16_t* W, bf16_t* act, int M, int F, int K,
                                const float* ssq, float eps) {
  constexpr int NPR = KQ == 2 ? MID_NPR : 1;
#define SP_GO(MTV)                                                                                                        \
  if constexpr ((!PACKED || MTV > KQ) && (MTV <= 10 || (KQ == 2 && PACKED))) {                                            \
    typedef GateupPipe<MTV, KQ, PACKED> P;                                                                                \
    hipLaunchKernelGGL((k_gemm_mid<MTV, CW, KQ, true, PACKED, true, P::KC, P::D, P::PF, NPR, P::WL>), dim3(n_cu),         \
                       dim3(64 * (CW * KQ + NPR)), 0, st, X, W, nullptr, act, M, F, K, 1, F / n_cu, ssq, eps);            \
  } else return hipErrorInvalidValue;
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

// Which plain products: all over row-major weights (1 to 160 rows, above).  In fragment order all of 65-160 rows, and of
// 17-64 rows those whose slices are at least 1024 deep: shorter ones (the 8B shape's O, four chunks) lose up to 8 % at 64
// rows, down gains (14336 and 28672 deep, 64 rows 28.1 / 26.8 and 83 / 77 us), and so do 12288-wide matrices (two
// layers at 64 rows 504 / 473).  Two 8B layers, the kernels before / with these (and gate/up of 17-32 rows in sp_gemm.hip's):
// 17 rows 217.4 / 218.7 us, 24 rows 220.6 / 219.6, 33 rows 230.5 / 228.8, 48 rows 237.1 / 233.4.  Up to 16 rows the kernels of
// one row tile stream weights in fragment order as fast without the loading waves.
bool sp_gemm_mid_takes(int M, int N, int K, bool packed, int n_cu) {
  if (M < 1 || M > 160 || N % 128 || K % MID_KC) return false;
  const MidCut cut = mid_cut(M, N, K, n_cu);
  return !packed || M > 64 || (M > 16 && cut.S >= 1 && K >= 1024 * cut.S);
}
// Which gate/up products: a CU's even share of 49-64 columns (four groups, two waves each; row-major from one row on,
// fragment order from three row tiles to 192 rows: 192 rows 57.7 us, in blocks of 128 rows 63.5; two row tiles sp_gemm.hip)
// or of 97-112 to 160 rows (seven groups, one wave each; row-major from one row on, a 70B layer at 1 / 16 rows 371 / 390 -> 293
// / 298 us; fragment order from two row tiles on, gate/up of the 70B shape at 128 rows 177.6 -> 149.4 us).
bool sp_gemm_mid_takes_gateup(int M, int F, int K, bool packed, int n_cu) {
  if (M < (packed ? 17 : 1) || M > 192 || K % 128 || n_cu < 1 || F % n_cu || (F / n_cu) % 8) return false;
  const int cpw = F / n_cu;
  return cpw > 48 && cpw <= 64 ? (packed ? M > 32 : M <= 160) : M <= 160 && cpw > 96 && cpw <= 112;
}

hipError_t sp_launch_gemm_mid(const bf16_t* X, const bf16_t* W, bool packed, float* out, int M, int N, int K, int n_cu,
                              int max_split, size_t part_capacity_floats, int* S_out, hipStream_t st, bool resident) {
  if (!sp_gemm_mid_takes(M, N, K, packed, n_cu)) return hipErrorInvalidValue;
  const MidCut cut = mid_cut(M, N, K, n_cu);
  const bool six = cut.cols == 96;
  const int tiles = N / cut.cols, chunks = K / MID_KC;
  int S = cut.S;
  if (S > max_split) S = max_split;
  // Two chunks a slice at least: one makes no use of the ring and costs twice the partial sums (2048 wide, four layers, 104 rows
  // 381 -> 367 us, row-major 64 rows 335 -> 320).
  if (S > chunks / 2) S = chunks > 1 ? chunks / 2 : 1;
  while (S > 1 && (size_t)S * M * N > part_capacity_floats) --S;
  if (S < 1) S = 1;
  if ((size_t)S * M * N > part_capacity_floats) return hipErrorInvalidValue;
  *S_out = S;
  const dim3 grid(tiles, S);
#define SP_GO(STRIPS, PK, NT, SH) return launch_plain<STRIPS, PK, NT, SH>(grid, st, X, W, out, M, N, K, S)
#define SP_BY_CACHE(STRIPS, PK, SH) { if (resident) SP_GO(STRIPS, PK, false, SH); else SP_GO(STRIPS, PK, true, SH); }
#define SP_BY_STRIPS(PK, SH) { if (six) SP_BY_CACHE(6, PK, SH) else SP_BY_CACHE(8, PK, SH) }
  if (!packed) SP_BY_STRIPS(false, false)
  if (K / S <= 2048) SP_BY_STRIPS(true, true)
  SP_BY_STRIPS(true, false)
#undef SP_BY_STRIPS
#undef SP_BY_CACHE
#undef SP_GO
}

hipError_t sp_launch_gemm_mid_gateup(const bf16_t* X, const bf16_t* W, bool packed, bf16_t* act, int M, int F, int K, int n_cu,
                                     const float* ssq, float eps, hipStream_t st) {
  if (!sp_gemm_mid_takes_gateup(M, F, K, packed, n_cu) || (ssq && M > 16)) return hipErrorInvalidValue;
  if (F / n_cu > 64)
    return packed ? launch_gateup<7, 1, true>(n_cu, st, X, W, act, M, F, K, ssq, eps) : launch_gateup<7, 1, false>(n_cu, st, X, W, act, M, F, K, ssq, eps);
  return packed ? launch_gateup<4, 2, true>(n_cu, st, X, W, act, M, F, K, ssq, eps) : launch_gateup<4, 2, false>(n_cu, st, X, W, act, M, F, K, ssq, eps);
}
