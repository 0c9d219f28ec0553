// Plain projections for one row tile (M <= 16: streaming steps of a few nodes, the single node after a stall), whole
// in one launch each.  A workgroup owns 16 output columns, or two strips of 16, and its waves cut the k range between them, so that the sums
// over k are complete inside the workgroup: there are no partial sums in memory, and what used to be a kernel of its own
// behind every split product -- RoPE and the cache append behind QKV, residual and RMSNorm behind O and down, the
// write-out behind the last layer -- is the epilogue here.
//
//   QKV:      q | k | v = scale[m] * sum_k X[m][k] W[n][k], rotated, to qbuf and to the node's cache rows
//   O, down:  h[m][n] += sum_k X[m][k] W[n][k];  X' = bf16(h * gain);  ssq[m][n / 16] = sum of the workgroup's h^2
//
// The RMSNorm of a row needs the whole row, which no workgroup sees: the producing kernel leaves h * gain and, per
// workgroup, the sum of its 16 squares, and the consuming kernel adds those up while its weights are on their way and
// multiplies the row's products by 1 / rms at the end (the norm is a factor per row, the projection is linear).
//
// With so few rows each weight is used once and the launch is bound by the weight stream and by its own start and end.
// A wave has D fragments of weights and of activations in flight: registers only, no LDS panel, no barrier before the
// waves are folded.  Measured at 6 rows, 8B shape, weights from HBM: QKV + RoPE 15.2 -> 13.0 us, O + residual + norm
// 12.1 -> 7.3 us, down + residual + norm 25.1 -> 20.0 us (before: split product and the kernel behind it); the step
// of four layers at a context of 32768 507 -> 465 us.  Four or sixteen waves, 4 to 16 fragments in flight and staggered starting
// steps are all within 2 % of this.
//
// Every workgroup reads all of X from L2, as much as it reads of the weights when all 16 rows are there, and that is
// what more rows cost (row-major rows, read in 64-byte pieces, 8192 x 28672: 71.5 us with one row, 95.4 with 16; beyond four
// rows they come in fragment order now, four 8B layers at 16 rows 426 -> 400 us a step).  Where N has 32 columns for each of the CUs a
// workgroup takes two strips of 16 and so half of that: 8192 x 28672 at 8 / 16 rows 75.6 -> 71.8 / 95.4 -> 80.8 us,
// 8192 x 8192 29.6 -> 27.2 / 35.4 -> 28.1, level up to 4 rows.  The two strips of all workgroups start 16 KB or a
// multiple apart in X, so these walk k from staggered starts (8192 x 8192: 31.1 -> 28.1 us; with one strip no gain).
#include "sp_launch.h"

#define FEW_WAVES 8        // waves per workgroup, each with an eighth of the k range
#define FEW_QKV 0
#define FEW_RESIDUAL 1
#define FEW_OUT 2          // residual of the last layer: the rows leave the stage

struct FewArgs {
  const bf16_t* X;         // [M][K], in fragment order or row-major
  const bf16_t* W;         // [N][K], row-major or in fragment order
  int M, N, K;
  bool frag;
  const float* ssq_in;     // [M][K / 16] sums of squares of the rows behind X (nullptr: X is normalised already)
  float eps;
  // QKV
  const RowInfo* rows;
  const float* cs;
  bf16_t* qbuf;
  KvGeom g;
  int layer, n_q, n_kv;
  // O, down
  float* h;                // [M][N]
  const bf16_t* gain;      // [N] gain of the norm that follows
  bf16_t* xn;              // [M][N], as X
  float* ssq_out;          // [M][N / 16]
  const AttnPlan* plan;    // FEW_OUT: x_out
};

template <int D, int NS, int MODE, bool PACKED, bool WNT, bool FRAG>
__global__ void __launch_bounds__(64 * FEW_WAVES) k_gemm_few(FewArgs a) {
  __shared__ __attribute__((aligned(16))) f32x4_t s_acc[NS][FEW_WAVES][64];
  __shared__ __attribute__((aligned(16))) float s_tot[16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kg = lane >> 4;
  const int K = a.K, M = a.M;
  const int n = (K >> 5) / FEW_WAVES;              // k steps of this wave, a multiple of D
  // QKV: a strip is columns t0 .. t0+7 of a head and their rotation partners t0+64 .. t0+71
  const bf16_t* w[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int bi = blockIdx.x * NS + i;
    const int wrow = MODE == FEW_QKV ? (bi >> 3) * 128 + (bi & 7) * 8 + (r & 7) + ((r & 8) << 3) : bi * 16 + r;
    w[i] = PACKED ? a.W + ((size_t)(wrow >> 4) * (K >> 5) + (size_t)wave * n) * 512 + (kg * 16 + (wrow & 15)) * 8
                           : a.W + (size_t)wrow * K + (size_t)wave * n * 32 + kg * 8;
  }
  const int b = blockIdx.x * NS + (wave < NS ? wave : 0), head = b >> 3, t0 = (b & 7) * 8;
  constexpr int WSTEP = PACKED ? 512 : 32;
  // rows past M repeat the last row and multiply into output rows that are never stored
  constexpr int XSTEP = FRAG ? 512 : 32;
  const bf16_t* x = a.X + (size_t)wave * n * XSTEP + (FRAG ? (kg * 16 + min(r, M - 1)) * 8 : min(r, M - 1) * K + kg * 8);
  u32x4_t wf[NS][D], xf[D];
  f32x4_t acc[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int rot = NS > 1 ? (int)(((blockIdx.x >> 3) * 2) % (unsigned)n) : 0;
#define SP_LD(j, S)                                                                             \
  {                                                                                             \
    const int p_ = NS > 1 && (S) + rot >= n ? (S) + rot - n : (S) + rot;                        \
    _Pragma("unroll") for (int i = 0; i < NS; ++i) {                                            \
      const u32x4_t* wp_ = reinterpret_cast<const u32x4_t*>(w[i] + (size_t)p_ * WSTEP);                 \
      wf[i][j] = WNT ? __builtin_nontemporal_load(wp_) : *wp_;                                  \
    }                                                                                           \
    xf[j] = *reinterpret_cast<const u32x4_t*>(x + p_ * XSTEP);                                 \
  }
#define SP_MM(j)                                                                                \
  _Pragma("unroll") for (int i = 0; i < NS; ++i)                                                \
  acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(&wf[i][j]),\
                                                *reinterpret_cast<const bf16x8_t*>(&xf[j]), acc[i], 0, 0, 0);
  // what the epilogue needs is asked for first: loads return in order, so nothing waits for it later
  RowSquares<64 * FEW_WAVES> sq;
  if (MODE == FEW_QKV && a.ssq_in) sq.load(a.ssq_in, K / 16, M);
  f32x4_t e0 = {0.f, 0.f, 0.f, 0.f}, e1 = {0.f, 0.f, 0.f, 0.f};   // h, or cos and sin
  uint2 gn = {0u, 0u};
  RowInfo ri;
  const int rc = min(r, M - 1);
  const int col = b * 16 + kg * 4;                 // O, down: this lane's four columns
  if (wave < NS) {
    if (MODE == FEW_QKV) {
      ri = a.rows[rc];
      const float* c = a.cs + (size_t)rc * 128 + t0 + (kg & 1) * 4;
      e0 = *reinterpret_cast<const f32x4_t*>(c);
      e1 = *reinterpret_cast<const f32x4_t*>(c + 64);
    } else {
      e0 = *reinterpret_cast<const f32x4_t*>(a.h + (size_t)rc * a.N + col);
      if (MODE == FEW_RESIDUAL) gn = *reinterpret_cast<const uint2*>(a.gain + col);
    }
  }

#pragma unroll
  for (int j = 0; j < D; ++j) SP_LD(j, j)
  for (int s = D; s < n; s += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      SP_MM(j)
      SP_LD(j, s + j)
    }
  }
#pragma unroll
  for (int j = 0; j < D; ++j) SP_MM(j)
#undef SP_LD
#undef SP_MM

#pragma unroll
  for (int i = 0; i < NS; ++i) s_acc[i][wave][lane] = acc[i];
  if (MODE == FEW_QKV && a.ssq_in) sq.post(a.ssq_in, K / 16, M, s_tot);
  __syncthreads();
  if (wave >= NS) return;
  // lane holds, for row r, columns 4 * kg .. + 3 of the workgroup's sixteen
  f32x4_t y = s_acc[wave][0][lane];
#pragma unroll
  for (int v = 1; v < FEW_WAVES; ++v) y += s_acc[wave][v][lane];
  if (MODE == FEW_QKV) {
    if (a.ssq_in) y *= rsqrtf(s_tot[rc] / (float)K + a.eps);
    f32x4_t o = y;
    if (head < a.n_q + a.n_kv) {                   // rotate: the partner columns are 32 lanes away
      f32x4_t p;
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = __shfl_xor(y[i], 32, 64);
      o = kg < 2 ? y * e0 - p * e1 : y * e0 + p * e1;
    }
    if (r >= M) return;
    const int t = t0 + (kg & 1) * 4 + (kg >> 1) * 64;
    bf16_t* dst;
    if (head < a.n_q) {
      dst = a.qbuf + ((size_t)r * a.n_q + head) * 128;
    } else {
      const bool is_k = head < a.n_q + a.n_kv;
      const int kvh = head - a.n_q - (is_k ? 0 : a.n_kv);
      const size_t slot = sp_phys_slot(a.g, ri.req, ri.base, ri.P + ri.node);
      dst = reinterpret_cast<bf16_t*>(a.g.kv + ((size_t)(a.layer * 2 + (is_k ? 0 : 1)) * a.n_kv + kvh) * a.g.plane_bytes +
                                      slot * a.g.row_bytes);
    }
    uint2 pk;
    pk.x = pack_bf16x2(o[0], o[1]);
    pk.y = pack_bf16x2(o[2], o[3]);
    *reinterpret_cast<uint2*>(dst + t) = pk;
  } else {
    y += e0;
    uint2 pk;
    if (MODE == FEW_OUT) {
      pk.x = pack_bf16x2(y[0], y[1]);
      pk.y = pack_bf16x2(y[2], y[3]);
      if (r < M) *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(a.plan->x_out) + (size_t)r * a.N + col) = pk;
      return;
    }
    const float s2 = quad_rows_sum((y[0] * y[0] + y[1] * y[1]) + (y[2] * y[2] + y[3] * y[3]));
    if (r >= M) return;
    if (kg == 0) a.ssq_out[r * (a.N / 16) + b] = s2;
    *reinterpret_cast<f32x4_t*>(a.h + (size_t)r * a.N + col) = y;
    pk.x = pack_bf16x2(y[0] * bf16_lo(gn.x), y[1] * bf16_hi(gn.x));
    pk.y = pack_bf16x2(y[2] * bf16_lo(gn.y), y[3] * bf16_hi(gn.y));
    *reinterpret_cast<uint2*>(a.xn + row_at(FRAG, r, col, a.N)) = pk;
  }
}

// Two strips per workgroup where that leaves a workgroup for each CU.  Not in QKV: 10240 columns make 320 workgroups, and
// an uneven last round (8192 deep, 1 / 16 rows: 31.0 -> 38.2 / 44.0 -> 46.7 us).
static bool two_strips(int N, int K, int n_cu) { return N % 32 == 0 && N >= 32 * n_cu && K % (256 * FEW_WAVES) == 0; }

// Where complete projections are taken: where they are faster than split products and the small kernels behind them, within
// some 3 %.  Measured with both over the widths 1024 to 16384, us a layer, complete / split:
// - Weights in fragment order, workgroups of O and down in whole rounds over the CUs (up to 4096 columns in strips of 16,
//   8192 in two strips): 1024 1 / 16 rows 33 / 38 and 38 / 44, 2048 45 / 53 and 54 / 61, 3072 56 / 66 and 66 / 74, 4096 90 / 99
//   and 100 / 106, 8192 1 / 12 / 16 rows 282 / 291, 293.8 / 296.0 and 295.1 / 297.1, 16384 967 / 981 and 16 rows 999 / 984.  An
//   uneven last round leaves most of the chip idle and more X to read: 4608 (288 workgroups) 1 / 4 / 16 rows 131 / 137 / 152
//   against 132 / 136 / 140, 5120 (320) d_ff = 13824 110 / 116 / 134 against 117 / 121 / 125, 27648 184 / 192 / 220 against 187
//   / 190 / 195, 7168 (448) 204 / 210 / 223 against 208 / 213 / 216: up to four rows there.
// - Row-major weights come in half lines here and in whole ones in the split products' kernel; what the complete ones save
//   behind the products makes up for that on narrow models: 1024 1 / 16 rows 37 / 44 and 44 / 48, 2048 54 / 61 and 64 / 67,
//   3072 1 / 8 / 10 rows 69 / 74, 76 / 78 and 79.8 / 78.7, 3584 1 / 4 / 8 rows 132 / 135, 140 / 138 and 142 / 138, 4096 1 / 8 / 16
//   rows 103.1 / 100.8, 106.8 / 105.2 and 112.6 / 106.0, 8192 one row 322 / 291.
// - One load in flight per wave does not stream: d_ff = 8960 and 11008 (35 and 43 k steps a wave) 54.5 / 51.1 and 106.6 /
//   106.0 with one row, 61.3 / 58.6 and 113.4 / 109.9 with 16.  Up to 1792 deep a wave has seven steps and it does not matter.
bool sp_few_takes(int M, int d, int dq, int F, bool packed, int n_cu) {
  auto streams = [](int K) { return K % (64 * FEW_WAVES) == 0 || K < 256 * FEW_WAVES; };
  auto whole_rounds = [&](int K) {
    const int wgs = d / (two_strips(d, K, n_cu) ? 32 : 16);
    return wgs <= n_cu || wgs % n_cu == 0;
  };
  if (M < 1 || M > 16 || !streams(d) || !streams(dq) || !streams(F)) return false;
  if (!packed) return d <= 16 * n_cu && M * d <= 4 * 8192;
  return whole_rounds(dq) && whole_rounds(F) ? M * d <= 12 * 8192 : M <= 4;
}

// Eight fragments in flight per wave; shapes whose k slices are shorter, or no multiple of that, take fewer.
template <int MODE, bool PACKED, bool WNT, bool FRAG>
static hipError_t launch_few_as(const FewArgs& a, int n_cu, hipStream_t st) {
  const int n = a.K / (32 * FEW_WAVES);
#define SP_GO(DV, NSV) hipLaunchKernelGGL((k_gemm_few<DV, NSV, MODE, PACKED, WNT, FRAG>), dim3(a.N / 16 / NSV), dim3(64 * FEW_WAVES), 0, st, a)
  if (MODE != FEW_QKV && two_strips(a.N, a.K, n_cu)) SP_GO(8, 2);
  else if (n % 8 == 0) SP_GO(8, 1);
  else if (n % 2 == 0) SP_GO(2, 1);
  else SP_GO(1, 1);
#undef SP_GO
  return hipGetLastError();
}
template <int MODE, bool PACKED, bool WNT>
static hipError_t launch_few(const FewArgs& a, int n_cu, hipStream_t st) {
  return a.frag ? launch_few_as<MODE, PACKED, WNT, true>(a, n_cu, st) : launch_few_as<MODE, PACKED, WNT, false>(a, n_cu, st);
}

hipError_t sp_launch_few_qkv(const bf16_t* X, bool frag, const bf16_t* W, bool packed, const float* ssq, float eps, const RowInfo* rows,
                             const float* cs, bf16_t* qbuf, KvGeom g, int layer, int M, int K, int n_q, int n_kv,
                             int n_cu, hipStream_t st) {
  if (M < 1 || M > 16 || K % 256 || g.row_bytes != 256) return hipErrorInvalidValue;
  FewArgs a = {};
  a.X = X; a.frag = frag; a.W = W; a.M = M; a.N = (n_q + 2 * n_kv) * 128; a.K = K; a.ssq_in = ssq; a.eps = eps;
  a.rows = rows; a.cs = cs; a.qbuf = qbuf; a.g = g; a.layer = layer; a.n_q = n_q; a.n_kv = n_kv;
  return packed ? launch_few<FEW_QKV, true, true>(a, n_cu, st) : launch_few<FEW_QKV, false, true>(a, n_cu, st);
}

hipError_t sp_launch_few_residual(const bf16_t* X, bool frag, const bf16_t* W, bool packed, bool resident, float* h, const bf16_t* gain,
                                  bf16_t* xn, float* ssq_out, int M, int N, int K, int n_cu,
                                  hipStream_t st) {
  if (M < 1 || M > 16 || K % 256 || N % 16) return hipErrorInvalidValue;
  FewArgs a = {};
  a.X = X; a.frag = frag; a.W = W; a.M = M; a.N = N; a.K = K; a.h = h; a.gain = gain; a.xn = xn; a.ssq_out = ssq_out;
  if (resident) return packed ? launch_few<FEW_RESIDUAL, true, false>(a, n_cu, st) : launch_few<FEW_RESIDUAL, false, false>(a, n_cu, st);
  return packed ? launch_few<FEW_RESIDUAL, true, true>(a, n_cu, st) : launch_few<FEW_RESIDUAL, false, true>(a, n_cu, st);
}

hipError_t sp_launch_few_out(const bf16_t* X, bool frag, const bf16_t* W, bool packed, const float* h, const AttnPlan* plan_dev, int M,
                             int N, int K, int n_cu, hipStream_t st) {
  if (M < 1 || M > 16 || K % 256 || N % 16) return hipErrorInvalidValue;
  FewArgs a = {};
  a.X = X; a.frag = frag; a.W = W; a.M = M; a.N = N; a.K = K; a.h = const_cast<float*>(h); a.plan = plan_dev;
  return packed ? launch_few<FEW_OUT, true, true>(a, n_cu, st) : launch_few<FEW_OUT, false, true>(a, n_cu, st);
}
