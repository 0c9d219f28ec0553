// bf16 products of few rows (M = tree nodes in flight) on the CDNA4 matrix cores, as far as no kernel of their own takes
// them: QKV, O and down over weights in fragment order up to 16 rows where sp_gemm_few.hip does not, and 17-64 rows with k
// slices too short for sp_gemm_mid.hip; gate/up of one row tile, of two where a CU's even share is 49-64 columns, and up to 128
// rows of widths that are no even share per CU; the output head and the logits, over weights in either order.  With so few
// rows every weight is used once, so the kernel is a weight streamer (decode is bound by loading parameters, Sec. 2.2): each wave pulls its 16 weight rows straight from HBM into registers in MFMA operand layout (one
// 16-byte load per lane per k-step, PF chunks ahead of the math), while the M x K activation panel -- shared by every wave
// -- is staged once per workgroup through LDS.  Up to 16 rows a workgroup is four waves over 64 columns (the panel is
// small, more workgroups stream better); from 17 rows on plain products take eight waves over 128 columns, one workgroup
// per CU, because the panel's way from L2 into the CU is then what the rows cost: it comes in fragment order, whose 1 KB
// loads that path moves at 120 B/ns per CU (16 rows of 64 bytes: 38).  The weights carry the non-temporal hint.
//
//   out[y][m][n] = sum_{k in slice y} X[m][k] * W[n][k]        (f32 partial sums)
//
// v_mfma_f32_16x16x32_bf16: A = 16 weight rows x 32 k (lane l: row l%16, k (l/16)*8..+8),
// B = 32 k x 16 activation rows (lane l: row l%16, same k), D[4*(l/16)+i][l%16].
#include "sp_launch.h"

// Tunables (defaults chosen by measurement on MI355X).
#ifndef SP_GEMM_KC_PLAIN
#define SP_GEMM_KC_PLAIN 128      // k per staged chunk (smaller LDS panel: three workgroups per CU)
#endif
#ifndef SP_GEMM_KC_GATEUP
#define SP_GEMM_KC_GATEUP 256
#endif
#ifndef SP_GEMM_PF
#define SP_GEMM_PF 2              // weight chunks in flight ahead of the math
#endif
// Workgroup shapes from 17 rows on, each measured against the four-wave 64-column workgroup it replaces (1 = on):
#ifndef SP_GEMM_PLAIN8
#define SP_GEMM_PLAIN8 1          // plain products, 17-64 rows: eight waves over 128 columns, one workgroup per CU
#endif
#ifndef SP_GEMM_PLAIN6
#define SP_GEMM_PLAIN6 1          // ... six waves over 96 columns where that divides the CUs evenly and 128 do not
#endif
#ifndef SP_GEMM_ARGMAX8
#define SP_GEMM_ARGMAX8 1         // the output head's top-column kernel in the eight-wave shape
#endif
#ifndef SP_GEMM_PF_EIGHT
#define SP_GEMM_PF_EIGHT SP_GEMM_PF   // the eight-wave plain kernels are faster with two
#endif
#ifndef SP_GEMM_NCG_PLAIN
#define SP_GEMM_NCG_PLAIN 4       // column groups (of 16 weight rows) per workgroup
#endif
#ifndef SP_GEMM_NCG_GATEUP
#define SP_GEMM_NCG_GATEUP 2
#endif
#ifndef SP_GEMM_ROT
// Plain products split over k, K up to 8192 (the QKV and O shapes): workgroups walk their k slice from
// different starting chunks.  At 32 and 64 rows 8192 x 8192 29.2 -> 24.8 and 31.0 -> 27.9 us, the other shapes
// within 1 %; nothing gained with K = 14336 or 28672 (down) and in gate/up over weights in fragment order: those keep
// the plain order.
#define SP_GEMM_ROT 1
#endif
#ifndef SP_GEMM_TARGET_WGS_ROWS
#define SP_GEMM_TARGET_WGS_ROWS 512   // split K until the grid has at most this many workgroups (two per CU)
#endif
#ifndef SP_GEMM_TARGET_WGS_ONE
#define SP_GEMM_TARGET_WGS_ONE 768    // ... or this many, for one row tile that those would load unevenly
#endif

// PACKED: the weights were re-laid at load time (sp_pack_weights) into MFMA fragment order --
// per strip of 16 rows, one contiguous 1 KB block per k-step of 32, lane-major -- so that every
// wave load is one contiguous kilobyte instead of sixteen 64-byte pieces.
// ARGMAX (output head of the last stage, Algorithm 1 "verify new token"): instead of the
// products, a workgroup leaves per row the largest of its 16*NCG columns and that column's
// index (the lowest one among equal maxima) as a (float, int) pair at out[(m * tiles + tile) * 2].
// LOGITS (lossy and stochastic verification): from two row tiles on the products of a workgroup's 128 columns lie together,
// [tile][m][column], stored non-temporally: written row by row the logits of 32 rows are pieces of 512 bytes half a megabyte
// apart and cost as much as 100 MB of weights (128256 x 4096, 32 rows: 187.2 us, in tiles 185.0, in tiles and non-temporal
// 178.7, without any stores 171.3).  Up to 16 rows what reads them gains more from finding them in L2 (3 to 14 rows, whole
// calls 0.4-1 % slower in tiles): row by row.  For a stochastic verification (stats given) a workgroup also leaves per row the
// maximum mx of its columns and the sum of exp((l - mx) * inv_T) over them as a float pair at stats[(m * tiles + tile) * 2].
// EVEN (gate/up of two row tiles over weights in fragment order): one workgroup per CU covers cpw = d_ff / CUs columns, a
// multiple of 8 in 49-64, in four groups of 16 and a last one of cpw - 48, by four groups times two k-halves of waves (the
// upper lanes of a short last group re-read its last row and their results are dropped).  With so few rows the loading waves
// of sp_gemm_mid.hip's kernel only take issue slots: gate/up of 17 / 32 rows 41.3 / 41.4 us here, 42.0 / 42.0 there, two 8B
// layers 216.6 / 222.1 and 219.4 / 223.4; from 33 rows on it is the other way round (43.0 / 42.2).
template <int MT, int NCG, bool GATEUP, int KC, int PF, bool PACKED, bool ARGMAX = false, int NWAVES = 4, bool WNT = true,
          bool LOGITS = false, bool FRAG = true, bool EVEN = false>
__global__ void __launch_bounds__(64 * NWAVES)
k_gemm_bf16(const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, float* __restrict__ out,
            bf16_t* __restrict__ act, int M, int N, int K, int chunks_total, int S, int rot = 0,
            const float* ssq = nullptr, float eps = 0.f, float* stats = nullptr, float inv_T = 0.f, int cpw = 0) {
  static_assert(!EVEN || (GATEUP && PACKED), "even share: gate/up over weights in fragment order");
  constexpr int NTH = 64 * NWAVES;
  constexpr int NKH = NWAVES / NCG;       // waves sharing a column group split each chunk's k-steps
  constexpr int KSTEPS = (KC / 32) / NKH;
  constexpr int NW = GATEUP ? 2 : 1;
  constexpr int ROWS = MT * 16;
  constexpr int UPT = KC * 2;             // 16-byte units of a row tile's chunk (KC / 32 fragment blocks, consecutive in X)
  constexpr int UNITS = MT * UPT;
  constexpr int XS = KC * 2 + 16, UPR = KC / 8;    // row-major X: padded LDS row in bytes, units per row
  constexpr int PASSES = (UNITS + NTH - 1) / NTH;  // the last staging pass may cover fewer units
  constexpr bool RAGGED_PASS = UNITS % NTH != 0;
  constexpr int NB = PF + 1;              // weight register buffers
  // two panels laid as X: in fragment order the fragment reads are conflict-free without padding
  constexpr int PANEL = FRAG ? UNITS * 16 : ROWS * XS;
  __shared__ __attribute__((aligned(16))) char lds[2 * PANEL];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int cg = wave % NCG, kh = wave / NCG;
  const int r = lane & 15, kg = lane >> 4;
  const int n0 = EVEN ? blockIdx.x * cpw + cg * 16 : blockIdx.x * (16 * NCG) + cg * 16;
  const int vr = EVEN ? min(16, cpw - cg * 16) : 16;     // valid columns of this wave's group (8 or 16)
  const int m_base = blockIdx.z * ROWS;
  const int c_begin = (int)(((long long)blockIdx.y * chunks_total) / S);
  const int c_end = (int)(((long long)(blockIdx.y + 1) * chunks_total) / S);

  // EVEN: a group starts at a multiple of 8, so its 16 rows may lie in two fragment blocks: per-lane row addresses
  const int wr = n0 + min(r, vr - 1);
  const bf16_t* w0 = EVEN ? W + ((size_t)(wr >> 4) * (K / 32) + kh * KSTEPS) * 512 + (kg * 16 + (wr & 15)) * 8
                   : PACKED ? W + ((size_t)(n0 / 16) * (K / 32) + kh * KSTEPS) * 512 + lane * 8
                            : W + (size_t)(n0 + r) * K + kg * 8 + kh * (KSTEPS * 32);
  const bf16_t* w1 = EVEN ? W + ((size_t)((N + wr) >> 4) * (K / 32) + kh * KSTEPS) * 512 + (kg * 16 + (wr & 15)) * 8
                   : PACKED ? W + ((size_t)((N + n0) / 16) * (K / 32) + kh * KSTEPS) * 512 + lane * 8     // the up rows
                            : W + (size_t)(N + n0 + r) * K + kg * 8 + kh * (KSTEPS * 32);
#define SP_WOFF(C, s) (PACKED ? ((size_t)(C) * (KC / 32) + (s)) * 512 : (size_t)(C)*KC + (s) * 32)
  // rot: workgroups start at different chunks of their k slice and wrap around, so that the workgroups of one
  // slice, whose weight rows lie a fixed distance apart, are not all at the same offset of their rows at the
  // same moment (the start moves with id / 8; id, id / 2, id / 4 and id / 16 measured worse).  The sum over k
  // is then taken in a different, still fixed, order per workgroup.
  const int c_n = c_end - c_begin;
  const int c_rot = rot && c_n > 1 ? (int)((blockIdx.x >> 3) % (unsigned)c_n) : 0;
#define SP_PC(C) ((C) + c_rot < c_end ? (C) + c_rot : (C) + c_rot - c_n)
  // row tiles past the last one repeat it, and of up to four tiles rows past M the last one (half of a nearly empty tile's
  // lines are then not asked for); what these multiply is never stored
  unsigned xo[PASSES];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int u = p * NTH + tid;
    const int tile = min((int)blockIdx.z * MT + u / UPT, (M - 1) >> 4);
    xo[p] = FRAG ? (unsigned)tile * (unsigned)(K * 16) + ((u % UPT & ~15) | (MT <= 4 ? min(u & 15, M - 1 - tile * 16) : u & 15)) * 8
                 : (unsigned)min(m_base + u / UPR, M - 1) * (unsigned)K + (u % UPR) * 8;
  }
  constexpr int XCHUNK = FRAG ? KC * 16 : KC;

  u32x4_t wb[NB][NW][KSTEPS];
  u32x4_t xnxt[PASSES];
  f32x4_t acc[NW][MT];
#pragma unroll
  for (int a = 0; a < NW; ++a)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[a][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

#define SP_LOAD_X(C)                                                                                   \
  _Pragma("unroll") for (int p = 0; p < PASSES; ++p) {                                                  \
    xnxt[p] = *reinterpret_cast<const u32x4_t*>(X + (size_t)SP_PC(C) * XCHUNK + xo[p]);                  \
  }
#define SP_STORE_X(BUF)                                                                                 \
  _Pragma("unroll") for (int p = 0; p < PASSES; ++p)                                                    \
      if (!RAGGED_PASS || p * NTH + tid < UNITS)                                                        \
        *reinterpret_cast<u32x4_t*>(&lds[(BUF) * PANEL + (FRAG ? (p * NTH + tid) * 16 : (p * NTH + tid) / UPR * XS + tid % UPR * 16)]) = xnxt[p];
  // Every weight is read once per launch: the loads carry the non-temporal hint (WNT), so the stream does not
  // push the activation panel (which every workgroup re-reads) out of L2 nor fill the Infinity Cache
  // (gate/up at 8 rows: 43.4 -> 38.8 us, at 64 rows: 50.7 -> 49.5 us).  The exception is a matrix the caller
  // wants to find in the Infinity Cache again at the next step: ordinary loads.
#define SP_LOAD_W(B, C)                                                                                 \
  _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s) {                                                  \
    const int pc_ = SP_PC(C);                                                                           \
    wb[B][0][s] = WNT ? __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(w0 + SP_WOFF(pc_, s))) \
                      : *reinterpret_cast<const u32x4_t*>(w0 + SP_WOFF(pc_, s));                         \
    if (NW == 2)                                                                                        \
      wb[B][NW - 1][s] = WNT ? __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(w1 + SP_WOFF(pc_, s))) \
                             : *reinterpret_cast<const u32x4_t*>(w1 + SP_WOFF(pc_, s));                  \
  }
  // One chunk C out of weight buffer B.  The activation panel of chunk C+1 was loaded to
  // registers one chunk earlier and goes to the other LDS buffer first; then the loads of
  // panel C+2 and of weight chunk C+PF are issued, and chunk C is multiplied.  A wave only
  // ever waits for loads that have had a whole chunk of math to arrive, and never for the
  // youngest weight loads (waits retire loads in issue order).
#define SP_CHUNK(B, C)                                                                                  \
  {                                                                                                     \
    const int c_ = (C);                                                                                 \
    const int buf = (c_ - c_begin) & 1;                                                                 \
    if (c_ + 1 < c_end) { SP_STORE_X(buf ^ 1) }                                                         \
    if (c_ + 2 < c_end) { SP_LOAD_X(c_ + 2) }                                                           \
    if (c_ + PF < c_end) { SP_LOAD_W((B + PF) % NB, c_ + PF) }                                          \
    _Pragma("unroll") for (int s = 0; s < KSTEPS; ++s) {                                                \
      _Pragma("unroll") for (int mt = 0; mt < MT; ++mt) {                                               \
        const bf16x8_t b = *reinterpret_cast<const bf16x8_t*>(                                          \
            &lds[buf * PANEL + (FRAG ? ((mt * (KC / 32) + kh * KSTEPS + s) * 64 + lane) * 16            \
                                     : (mt * 16 + r) * XS + ((kh * KSTEPS + s) * 32 + kg * 8) * 2)]);   \
        _Pragma("unroll") for (int a = 0; a < NW; ++a) acc[a][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16( \
            *reinterpret_cast<const bf16x8_t*>(&wb[B][a][s]), b, acc[a][mt], 0, 0, 0);                  \
      }                                                                                                 \
    }                                                                                                   \
    __syncthreads();                                                                                    \
  }

  // one row tile of gate/up: the rows may come without their RMSNorm, whose scale is then a factor of the products
  constexpr bool SCALED = GATEUP && MT == 1;
  RowSquares<NTH> sq;
  if (SCALED && ssq) sq.load(ssq, K / 16, M);
  if (c_begin < c_end) {
    SP_LOAD_X(c_begin)
    SP_LOAD_W(0, c_begin)
    if (PF >= 2 && c_begin + 1 < c_end) { SP_LOAD_W(1 % NB, c_begin + 1) }
    if (PF >= 3 && c_begin + 2 < c_end) { SP_LOAD_W(2 % NB, c_begin + 2) }
    SP_STORE_X(0)
    if (c_begin + 1 < c_end) { SP_LOAD_X(c_begin + 1) }
  }
  __syncthreads();
  for (int c = c_begin; c < c_end; c += NB) {
    SP_CHUNK(0, c)
    if (NB >= 2 && c + 1 < c_end) SP_CHUNK(1 % NB, c + 1)
    if (NB >= 3 && c + 2 < c_end) SP_CHUNK(2 % NB, c + 2)
    if (NB >= 4 && c + 3 < c_end) SP_CHUNK(3 % NB, c + 3)
  }
  static_assert(PF >= 1 && PF <= 3, "weight chunks in flight");
#undef SP_CHUNK
#undef SP_LOAD_W
#undef SP_STORE_X
#undef SP_LOAD_X
#undef SP_PC
#undef SP_WOFF

  float* s_tot = reinterpret_cast<float*>(lds) + (sizeof(lds) / 4 - 16);      // behind the fold's floats
  if (SCALED && ssq) sq.post(ssq, K / 16, M, s_tot);
  if (NKH == 2) {       // fold the two k-halves of a column group together through LDS
    static_assert(!SCALED || (NCG * NW * MT * 64 * 4 + 16) * 4 <= (int)sizeof(lds), "fold and row sums side by side");
    float* red = reinterpret_cast<float*>(lds);
    if (kh == 1) {
#pragma unroll
      for (int a = 0; a < NW; ++a)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          *reinterpret_cast<f32x4_t*>(red + (((cg * NW + a) * MT + mt) * 64 + lane) * 4) = acc[a][mt];
    }
    __syncthreads();
    if (kh == 1) return;
#pragma unroll
    for (int a = 0; a < NW; ++a)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[a][mt] += *reinterpret_cast<const f32x4_t*>(red + (((cg * NW + a) * MT + mt) * 64 + lane) * 4);
  }

  // lane holds, for activation row m = mt*16 + l%16, output columns n0 + 4*(l/16) + 0..3
  const int ncol = n0 + 4 * kg;
  if (EVEN && 4 * kg >= vr) return;       // columns past a short last group
  if (ARGMAX) {
    static_assert(!ARGMAX || (NKH == 1 && !GATEUP), "one wave per column group");
    float* s_val = reinterpret_cast<float*>(lds);          // [NCG][ROWS]; the panels are no longer read
    int* s_idx = reinterpret_cast<int*>(s_val + NCG * ROWS);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float bv = acc[0][mt][0];
      int bi = ncol;
#pragma unroll
      for (int i = 1; i < 4; ++i)
        if (acc[0][mt][i] > bv) { bv = acc[0][mt][i]; bi = ncol + i; }
#pragma unroll
      for (int off = 16; off <= 32; off <<= 1) {                  // the four lanes that hold the row
        const float ov = __shfl_xor(bv, off, 64);
        const int oi = __shfl_xor(bi, off, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
      }
      if (kg == 0) { s_val[cg * ROWS + mt * 16 + r] = bv; s_idx[cg * ROWS + mt * 16 + r] = bi; }
    }
    __syncthreads();
    const int m = m_base + tid;
    if (tid < ROWS && m < M) {
      float bv = s_val[tid];
      int bi = s_idx[tid];
#pragma unroll
      for (int c = 1; c < NCG; ++c)                               // ascending columns: ties keep the lower one
        if (s_val[c * ROWS + tid] > bv) { bv = s_val[c * ROWS + tid]; bi = s_idx[c * ROWS + tid]; }
      float* o = out + ((size_t)m * gridDim.x + blockIdx.x) * 2;
      o[0] = bv;
      reinterpret_cast<int*>(o)[1] = bi;
    }
    return;
  }
  if (LOGITS && stats) {
    static_assert(!LOGITS || (NKH == 1 && !GATEUP && !ARGMAX), "one wave per column group");
    float* s_mx = reinterpret_cast<float*>(lds);           // [NCG][ROWS]; the panels are no longer read
    float* s_z = s_mx + NCG * ROWS;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const f32x4_t v = acc[0][mt];
      const float mx = quad_rows_max(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
      const float ref = mx == -INFINITY ? 0.f : mx;               // a piece without a finite value adds nothing
      float z = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) z += expf((v[i] - ref) * inv_T);
      z = quad_rows_sum(z);
      if (kg == 0) { s_mx[cg * ROWS + mt * 16 + r] = mx; s_z[cg * ROWS + mt * 16 + r] = z; }
    }
    __syncthreads();
    if (tid < ROWS && m_base + tid < M) {
      float mx = s_mx[tid];
#pragma unroll
      for (int c = 1; c < NCG; ++c) mx = fmaxf(mx, s_mx[c * ROWS + tid]);
      float z = 0.f;
#pragma unroll
      for (int c = 0; c < NCG; ++c) {
        const float pm = s_mx[c * ROWS + tid];
        z += s_z[c * ROWS + tid] * (pm == mx || pm == -INFINITY ? 1.f : expf((pm - mx) * inv_T));
      }
      *reinterpret_cast<float2*>(stats + ((size_t)(m_base + tid) * gridDim.x + blockIdx.x) * 2) = make_float2(mx, z);
    }
  }
  float row_scale = 1.f;
  if (SCALED && ssq) {
    if (NKH != 2) __syncthreads();      // (the fold of the k-halves has passed a barrier)
    row_scale = rsqrtf(s_tot[min(r, M - 1)] / (float)K + eps);
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int m = m_base + mt * 16 + r;
    if (m >= M) continue;
    if (GATEUP) {
      float o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float gte = SCALED ? acc[0][mt][i] * row_scale : acc[0][mt][i];
        const float up = SCALED ? acc[NW - 1][mt][i] * row_scale : acc[NW - 1][mt][i];
        o[i] = gte / (1.f + __expf(-gte)) * up;
      }
      uint2 pk;
      pk.x = pack_bf16x2(o[0], o[1]);
      pk.y = pack_bf16x2(o[2], o[3]);
      *reinterpret_cast<uint2*>(act + row_at(FRAG, m, ncol, N)) = pk;
    } else if (LOGITS && NCG == 8) {
      __builtin_nontemporal_store(acc[0][mt], reinterpret_cast<f32x4_t*>(out + ((size_t)blockIdx.x * M + m) * (16 * NCG) + cg * 16 + 4 * kg));
    } else {
      float* o = out + ((size_t)blockIdx.y * M + m) * N + ncol;
      *reinterpret_cast<f32x4_t*>(o) = acc[0][mt];
    }
  }
}

// ---- launchers -------------------------------------------------------------------
// Rows beside row-major weights (the output head and the logits; gate/up takes them as the call's other products do) lie
// row-major, whatever their number: as many 64-byte pieces of the weights are on their way as L2 takes, and the panel of
// sixteen rows in fragment order came on top (128256 x 4096, 1 / 8 / 48 rows: 212 / 218 / 250 us, in fragment order 222 / 224 /
// 257).
// Up to 64 rows run as one block of MT = ceil(M/16) tiles; more rows (gate/up of other widths, the output head) run in
// blocks of 128 (MT = 8, always with the 128-wide chunk so that the two LDS panels fit), each block streaming the weights
// once.
// staggered starting chunks: plain products that are split over k, K up to 8192 (see SP_GEMM_ROT)
static inline int rot_for(int S, int K) { return (SP_GEMM_ROT && S > 1 && K <= 8192) ? 1 : 0; }

template <int NCG, bool GATEUP, int KCV, bool PACKED, bool ARGMAX = false>
static hipError_t launch_mt(int MT, dim3 grid, hipStream_t st, const bf16_t* X, const bf16_t* W, float* out,
                            bf16_t* act, int M, int N, int K, int S, const float* ssq = nullptr, float eps = 0.f, bool frag = true) {
#define SP_GO(MTV, KCX)                                                                                        \
  hipLaunchKernelGGL((k_gemm_bf16<MTV, NCG, GATEUP, KCX, SP_GEMM_PF, PACKED, ARGMAX, 4, true, false, GATEUP || PACKED>), grid, dim3(256), 0, st, X, \
                     W, out, act, M, N, K, K / KCX, S, (!GATEUP && !ARGMAX) ? rot_for(S, K) : 0, ssq, eps)
  if constexpr (!ARGMAX && (GATEUP ? NCG != 4 : PACKED))
    if (!frag) {
      hipLaunchKernelGGL((k_gemm_bf16<1, NCG, GATEUP, KCV, SP_GEMM_PF, PACKED, ARGMAX, 4, true, false, false>), grid, dim3(256), 0,
                         st, X, W, out, act, M, N, K, K / KCV, S, GATEUP ? 0 : rot_for(S, K), ssq, eps);
      return hipGetLastError();
    }
  if (!ARGMAX && MT == 4 && GATEUP && NCG == 4) {      // the 64 + 64 column gate/up workgroup at 49-64 rows
    hipLaunchKernelGGL((k_gemm_bf16<4, 4, true, 128, SP_GEMM_PF, PACKED, false>), grid, dim3(256), 0, st, X, W, out, act, M, N, K, K / 128, S);
    return hipGetLastError();
  }
  switch (MT) {
    case 1: SP_GO(1, KCV); break;
    case 2: SP_GO(2, KCV); break;
    case 3: SP_GO(3, KCV); break;
    case 4: SP_GO(4, KCV); break;
    default:
      if (ARGMAX) SP_GO(8, 128);
      else if (GATEUP && NCG == 4)
        hipLaunchKernelGGL((k_gemm_bf16<8, 4, true, 128, SP_GEMM_PF, PACKED, false>), grid, dim3(256), 0, st, X, W, out, act,
                           M, N, K, K / 128, S);
      else if (GATEUP) SP_GO(8, 128);
      else return hipErrorInvalidValue;               // plain products of eight row tiles: not in these workgroups
      break;
  }
#undef SP_GO
  return hipGetLastError();
}
// columns one workgroup covers
static inline int tile_cols(int MT, bool gateup) { return 16 * (gateup ? SP_GEMM_NCG_GATEUP : SP_GEMM_NCG_PLAIN); }

static inline void row_blocks(int M, int* MT, int* mblocks) {
  if (M <= 64) { *MT = (M + 15) / 16; *mblocks = 1; }
  else { *MT = 8; *mblocks = (M + 127) / 128; }
}

hipError_t sp_launch_gemm_bf16(const bf16_t* X, const bf16_t* W, bool packed, float* out, int M, int N, int K,
                               int max_split, size_t part_capacity_floats, int* S_out, hipStream_t st, bool resident, bool frag) {
  const int MT = (M + 15) / 16;
  // 17-64 rows: workgroups of eight waves over 128 columns, one per CU -- the same waves per CU as two
  // four-wave workgroups of 64 columns, but the panel slice is staged once for all eight
  const bool eight = SP_GEMM_PLAIN8 && N % 128 == 0 && MT >= 2;
  // ... or six waves over 96 columns where that divides the CUs evenly and 128 columns do not (N = 6144 on 256 CUs:
  // 64 tiles x 4 slices of equal length instead of 48 x 5 of 6 or 7 chunks)
  const bool six = SP_GEMM_PLAIN6 && eight && N % 96 == 0 && (SP_GEMM_TARGET_WGS_ROWS / 2) % (N / 128) != 0 &&
                   (SP_GEMM_TARGET_WGS_ROWS / 2) % (N / 96) == 0;
  const int TILE = six ? 96 : eight ? 128 : 16 * SP_GEMM_NCG_PLAIN;
  if (M < 1 || M > 64 || (packed ? !frag && M > 8 : frag) || N % TILE || K % SP_GEMM_KC_PLAIN || K % 128) return hipErrorInvalidValue;
  const int chunks = K / SP_GEMM_KC_PLAIN;
  const int tiles = N / TILE;
  // Enough workgroups to keep every CU streaming, within the partial-sum buffer.  Every slice costs M*N*4 bytes
  // written here and read again by the kernel that folds them, which outweighs a finer split: at most two
  // workgroups per CU (measured on the whole 64-row step: 0.608 ms against 0.617 ms with three; a count between
  // two and three per CU, which leaves the CUs unevenly loaded, 0.638 ms; two waves per column group with half
  // the slices again: 0.612 ms).
  int S = (eight ? SP_GEMM_TARGET_WGS_ROWS / 2 : SP_GEMM_TARGET_WGS_ROWS) / tiles;
  // One row tile, whose partial sums are small: three workgroups per CU where two per CU would be an uneven round (12288
  // columns: 192 tiles x 4 instead of x 2; a layer with those in O and down at 8 / 16 rows 461.5 -> 456.5 and 473 -> 463 us, four
  // with those in QKV at one row 213 -> 202.5).  Not throughout: 7168 and 5120 columns in 112 x 7 and 80 x 10 workgroups, a few
  // more than three per CU, 156 -> 165 us at one row.
  if (MT == 1 && S >= 1 && 4 * S * tiles <= 3 * SP_GEMM_TARGET_WGS_ROWS) S = (SP_GEMM_TARGET_WGS_ONE + tiles - 1) / tiles;
  if (S > max_split) S = max_split;
  if (S > chunks) S = chunks;
  while (S > 1 && (size_t)S * M * N > part_capacity_floats) --S;
  if (S < 1) S = 1;
  if ((size_t)S * M * N > part_capacity_floats) return hipErrorInvalidValue;
  *S_out = S;
  const dim3 grid(tiles, S);
  if (six) {
#define SP_GO6(MTV, PK)                                                                                          \
  hipLaunchKernelGGL((k_gemm_bf16<MTV, 6, false, SP_GEMM_KC_PLAIN, SP_GEMM_PF, PK, false, 6, true, false, PK>), grid, dim3(384), 0, \
                     st, X, W, out, nullptr, M, N, K, K / SP_GEMM_KC_PLAIN, S, rot_for(S, K))
    if (packed) { if (MT == 2) SP_GO6(2, true); else if (MT == 3) SP_GO6(3, true); else SP_GO6(4, true); }
    else { if (MT == 2) SP_GO6(2, false); else if (MT == 3) SP_GO6(3, false); else SP_GO6(4, false); }
#undef SP_GO6
    return hipGetLastError();
  }
  if (eight) {
#define SP_GO8(MTV, PK)                                                                                          \
  if (PK && resident)                                                                                            \
    hipLaunchKernelGGL((k_gemm_bf16<MTV, 8, false, SP_GEMM_KC_PLAIN, SP_GEMM_PF_EIGHT, true, false, 8, false>),  \
                       grid, dim3(512), 0, st, X, W, out, nullptr, M, N, K, K / SP_GEMM_KC_PLAIN, S, rot_for(S, K)); \
  else                                                                                                           \
  hipLaunchKernelGGL((k_gemm_bf16<MTV, 8, false, SP_GEMM_KC_PLAIN, SP_GEMM_PF_EIGHT, PK, false, 8, true, false, PK>), grid, dim3(512), 0, \
                     st, X, W, out, nullptr, M, N, K, K / SP_GEMM_KC_PLAIN, S, rot_for(S, K))
    if (packed) { if (MT == 2) SP_GO8(2, true); else if (MT == 3) SP_GO8(3, true); else SP_GO8(4, true); }
    else { if (MT == 2) SP_GO8(2, false); else if (MT == 3) SP_GO8(3, false); else SP_GO8(4, false); }
#undef SP_GO8
    return hipGetLastError();
  }
  // One row tile of a matrix that is to stay in the Infinity Cache: ordinary weight loads from 9 rows on (two layers of 4608 and
  // 5120 columns at 16 rows 282.4 -> 280.5 and 251.7 -> 249.3 us; of 4096 columns with d_ff = 11008 at 9 / 16 rows 203.9 -> 206.7 and
  // 211.0 -> 209.8); with fewer it is level (4608 wide, 8 rows 144.5 -> 146.5).
  if (resident && packed && M > 8) {
    hipLaunchKernelGGL((k_gemm_bf16<1, SP_GEMM_NCG_PLAIN, false, SP_GEMM_KC_PLAIN, SP_GEMM_PF, true, false, 4, false>),
                       grid, dim3(256), 0, st, X, W, out, nullptr, M, N, K, K / SP_GEMM_KC_PLAIN, S, rot_for(S, K));
    return hipGetLastError();
  }
  if (packed) return launch_mt<SP_GEMM_NCG_PLAIN, false, SP_GEMM_KC_PLAIN, true>(MT, grid, st, X, W, out, nullptr, M, N, K, S, nullptr, 0.f, frag);
  return launch_mt<SP_GEMM_NCG_PLAIN, false, SP_GEMM_KC_PLAIN, false>(MT, grid, st, X, W, out, nullptr, M, N, K, S);
}

hipError_t sp_launch_gemm_gateup_bf16(const bf16_t* X, bool frag, const bf16_t* W, bool packed, bf16_t* act, int M, int F,
                                      int K, int n_cu, const float* ssq, float eps, hipStream_t st) {
  int MT, mblocks;
  row_blocks(M, &MT, &mblocks);
  if ((ssq || !frag) && MT != 1) return hipErrorInvalidValue;
  if (M < 1 || F % 64 || K % SP_GEMM_KC_GATEUP || K % 128) return hipErrorInvalidValue;
  // two row tiles and a CU's even share of 49-64 columns: one workgroup of eight waves per CU (see EVEN)
  if (packed && MT == 2 && n_cu > 0 && F % n_cu == 0 && (F / n_cu) % 8 == 0 && F / n_cu > 48 && F / n_cu <= 64) {
    hipLaunchKernelGGL((k_gemm_bf16<2, 4, true, SP_GEMM_KC_GATEUP, SP_GEMM_PF, true, false, 8, true, false, true, true>), dim3(n_cu), dim3(512), 0, st,
                       X, W, nullptr, act, M, F, K, K / SP_GEMM_KC_GATEUP, 1, 0, nullptr, 0.f, nullptr, 0.f, F / n_cu);
    return hipGetLastError();
  }
  // From 49 rows on: 64 gate + 64 up columns per workgroup (four column groups, 128-k chunks) where that
  // still gives every CU a workgroup, so that the staged panel is at most as large as the weights it meets
  // (70B shape: gate/up 193.6 -> 179.3 us at 64 rows, 252 -> 212 us at 128 rows); else 32 + 32 columns.  With
  // d_ff = 14336 the wider workgroups number 224 and run level with the 448 narrow ones (53.2 against 53.9 us).
  if ((MT == 8 || MT == 4) && F / 64 * mblocks >= 256) {
    const dim3 grid(F / 64, 1, mblocks);
    if (packed) return launch_mt<4, true, SP_GEMM_KC_GATEUP, true>(MT, grid, st, X, W, nullptr, act, M, F, K, 1);
    return launch_mt<4, true, SP_GEMM_KC_GATEUP, false>(MT, grid, st, X, W, nullptr, act, M, F, K, 1);
  }
  const int TILE = tile_cols(MT, true);
  const dim3 grid(F / TILE, 1, mblocks);
  if (packed) return launch_mt<SP_GEMM_NCG_GATEUP, true, SP_GEMM_KC_GATEUP, true>(MT, grid, st, X, W, nullptr, act, M, F, K, 1, ssq, eps, frag);
  return launch_mt<SP_GEMM_NCG_GATEUP, true, SP_GEMM_KC_GATEUP, false>(MT, grid, st, X, W, nullptr, act, M, F, K, 1, ssq, eps, frag);
}

// Output head: per row the top column of every 64-column tile, as (value, index) pairs
// pairs[(m * tiles + tile) * 2]; *tiles_out = V / 64.  One pass over the vocabulary matrix.
hipError_t sp_launch_gemm_argmax_bf16(const bf16_t* X, const bf16_t* W, bool packed, float* pairs, int M, int V, int K,
                                      size_t pair_capacity_floats, int* tiles_out, hipStream_t st) {
  static_assert(SP_GEMM_NCG_PLAIN == 4, "the top-column epilogue needs one wave per column group");
  int MT, mblocks;
  row_blocks(M, &MT, &mblocks);
  // 17-64 rows: eight waves over 128 columns share one staged panel, as in the plain projections
  const bool eight = SP_GEMM_ARGMAX8 && MT >= 2 && MT <= 4 && V % 128 == 0 && SP_GEMM_KC_PLAIN == 128;
  const int TILE = eight ? 128 : 16 * SP_GEMM_NCG_PLAIN;
  if (M < 1 || V % TILE || K % SP_GEMM_KC_PLAIN || K % 128) return hipErrorInvalidValue;
  const int tiles = V / TILE;
  if ((size_t)M * tiles * 2 > pair_capacity_floats) return hipErrorInvalidValue;
  *tiles_out = tiles;
  const dim3 grid(tiles, 1, mblocks);
  if (eight) {
#define SP_GOA(MTV, PK)                                                                                        \
  hipLaunchKernelGGL((k_gemm_bf16<MTV, 8, false, 128, SP_GEMM_PF, PK, true, 8, true, false, PK>), grid, dim3(512), 0, st, X, W, \
                     pairs, nullptr, M, V, K, K / 128, 1)
    if (packed) { if (MT == 2) SP_GOA(2, true); else if (MT == 3) SP_GOA(3, true); else SP_GOA(4, true); }
    else { if (MT == 2) SP_GOA(2, false); else if (MT == 3) SP_GOA(3, false); else SP_GOA(4, false); }
#undef SP_GOA
    return hipGetLastError();
  }
  if (packed) return launch_mt<SP_GEMM_NCG_PLAIN, false, SP_GEMM_KC_PLAIN, true, true>(MT, grid, st, X, W, pairs, nullptr, M, V, K, 1);
  return launch_mt<SP_GEMM_NCG_PLAIN, false, SP_GEMM_KC_PLAIN, false, true>(MT, grid, st, X, W, pairs, nullptr, M, V, K, 1);
}

// Logits (M <= 64, no split), [M][V] or as logits_lie says, and, where stats is given, the statistics of every tile of
// *tile_cols columns: stats[(m * V / *tile_cols + tile) * 2] = (maximum, sum of exp((l - maximum) * inv_T)).
hipError_t sp_launch_gemm_logits_bf16(const bf16_t* X, const bf16_t* W, bool packed, float* logits, float* stats, float inv_T,
                                      int M, int V, int K, int* tile_cols, hipStream_t st) {
  const int MT = (M + 15) / 16;
  const bool eight = MT >= 2 && V % 128 == 0;           // shapes as in the plain projections
  const int TILE = eight ? 128 : 64;
  if (M < 1 || M > 64 || V % TILE || K % SP_GEMM_KC_PLAIN || K % 128) return hipErrorInvalidValue;
  *tile_cols = TILE;
  const dim3 grid(V / TILE);
#define SP_GOL(MTV, NCGV, PK)                                                                                          \
  hipLaunchKernelGGL((k_gemm_bf16<MTV, NCGV, false, SP_GEMM_KC_PLAIN, SP_GEMM_PF, PK, false, NCGV, true, true, PK>), \
                     grid, dim3(64 * NCGV), 0, st, X, W, logits, nullptr, M, V, K, K / SP_GEMM_KC_PLAIN, 1, 0, nullptr, 0.f, stats, inv_T)
#define SP_GOT(NCGV, PK) if (MT == 2) SP_GOL(2, NCGV, PK); else if (MT == 3) SP_GOL(3, NCGV, PK); else SP_GOL(4, NCGV, PK)
  if (eight) { if (packed) { SP_GOT(8, true); } else { SP_GOT(8, false); } }
  else if (MT == 1) { if (packed) SP_GOL(1, 4, true); else SP_GOL(1, 4, false); }
  else { if (packed) { SP_GOT(4, true); } else { SP_GOT(4, false); } }
#undef SP_GOT
#undef SP_GOL
  return hipGetLastError();
}

// Re-lays a [N][K] row-major bf16 matrix into MFMA fragment order: 16-byte unit u of the output
// holds W[strip*16 + u%16][kstep*32 + ((u/16)%4)*8 .. +8] with u/64 = strip*(K/32) + kstep.
__global__ void k_pack_weights(const u32x4_t* __restrict__ in, u32x4_t* __restrict__ out, int N, int K) {
  const size_t units = (size_t)N * K / 8;
  for (size_t u = (size_t)blockIdx.x * blockDim.x + threadIdx.x; u < units; u += (size_t)gridDim.x * blockDim.x) {
    const size_t blk = u >> 6;
    const int lane = (int)(u & 63);
    const size_t strip = blk / (K / 32), ks = blk - strip * (K / 32);
    const size_t n = strip * 16 + (lane & 15), k = ks * 32 + (lane >> 4) * 8;
    out[u] = in[(n * K + k) / 8];
  }
}

hipError_t sp_launch_pack_weights(const void* in, void* out, int N, int K, hipStream_t st) {
  if (N % 16 || K % 32 || in == out) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pack_weights, dim3(4096), dim3(256), 0, st, (const u32x4_t*)in, (u32x4_t*)out, N, K);
  return hipGetLastError();
}
