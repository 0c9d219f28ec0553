// float32 kernels: products on the matrix cores (v_mfma_f32_16x16x4_f32: float32 operands and accumulation) and tree
// attention by four waves per (row, query head).  At the sizes a float32 stage is run with (d = 256, some 16 nodes) a
// launch is a chain of memory latencies, so what counts is how few of them stand in a row: the waves of a workgroup cut
// the k range (or the cache slots) between them and have several loads each in flight, and are folded through LDS.
// Measured on the two-layer d = 256 stage, 16 nodes, context 128 (one thread column per output and one wave per row
// and head before): products of 256 and 688 k 12.0 and 18.3 -> 4.6 and 4.7 us, attention 27.8 -> 5.5 us.  For the same
// reason a layer is five launches: RMSNorm, rotation, cache append, residual and write-out are prologues and epilogues of
// the products: 2 layers, 16 nodes, a call 80 -> 70 us (70.1 -> 60.7 back to back), 64 nodes 104 -> 94.
#include <type_traits>

#include "sp_launch.h"

#define F_WAVES 8

// What becomes of the products y[m][n] = sum_k X[m][k] W[n][k]:
enum F32Mode {
  F_PLAIN,      // out = y
  F_QKV,        // X = rmsnorm(h): queries and keys rotated, values copied; queries to out [M][n_q * d_head], the rest to the cache
  F_GATEUP,     // X = rmsnorm(h): out = silu(X Wg^T) * (X Wu^T), W = [N gate rows ; N up rows]
  F_RESIDUAL,   // out += y (out is h; X is another buffer)
  F_OUT         // the plan's x_out = h + y (out is h)
};
struct F32Args {
  const float* gain; float eps;                                                              // F_QKV, F_GATEUP
  const RowInfo* rows; const float* cs; KvGeom g; int layer, n_q, n_kv, d_head;              // F_QKV
  const AttnPlan* plan;                                                                      // F_OUT
};

// RMSNorm as a prologue: rows come as h[m][k] * gain[k], their squares are summed on the way (every workgroup reads whole
// rows, each of its waves and lanes another part), and 1 / sqrt(mean + eps) multiplies the finished sums.  Scale and residual
// are applied to the sums in 64 bits, so that a product is rounded as often as behind a norm of its own.
// F_QKV: the 16 columns of a workgroup are eight rotation pairs, t0 .. t0 + 7 and the same d_head / 2 further on, so a
// lane's partner value is its neighbour's in lane ^ 32.
// A workgroup covers 16 columns and 16 * MT rows.  A lane's 16-byte piece holds four consecutive k of its row; MFMA i of
// the four takes element i of every lane's piece, so lane group kg contributes k = 16 * step + 4 * kg + i on both sides.
template <int MT, int MODE>
__global__ void __launch_bounds__(64 * F_WAVES) k_gemm_f32(const float* __restrict__ X, const float* __restrict__ W,
                                                           float* __restrict__ out, int M, int N, int K, F32Args fa) {
  constexpr bool GATEUP = MODE == F_GATEUP, NORM = MODE == F_QKV || MODE == F_GATEUP;
  constexpr int NS = GATEUP ? 2 : 1;
  // 16-byte pieces of every operand in flight per lane: four; two in the largest gate/up, which spills with four, and in that of
  // one row tile, where two leave 128 registers and so two workgroups to a CU (4096 x 28672, one row, 113 -> 103 us)
  constexpr int F_D = GATEUP && MT != 2 ? 2 : 4;
  __shared__ __attribute__((aligned(16))) f32x4_t s_acc[F_WAVES][NS * MT][64];
  __shared__ double s_ss[F_WAVES][NORM ? MT : 1][16];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int r = lane & 15, kg = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * (16 * MT);
  const int pieces = K / 4, steps = (pieces + 3) / 4;
  const int s_begin = steps * wave / F_WAVES, s_end = steps * (wave + 1) / F_WAVES;
  // rows past the end repeat the last one; their products are not stored
  const float* w[NS];
  const float* x[MT];
#pragma unroll
  for (int a = 0; a < NS; ++a) w[a] = W + (size_t)(a * N + min(n0 + r, N - 1)) * K;
  int head = 0, t0 = 0, half = 0;
  if constexpr (MODE == F_QKV) {
    half = fa.d_head >> 1;
    head = n0 / fa.d_head;
    t0 = (n0 - head * fa.d_head) >> 1;
    w[0] = W + (size_t)(head * fa.d_head + t0 + (r & 7) + (r >> 3) * half) * K;
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) x[mt] = X + (size_t)min(m0 + mt * 16 + r, M - 1) * K;
  // What the finishing waves need is asked for first: the largest workgroups are alone on their CUs, and nothing would cover
  // the wait (d = 256, 1536 columns, 64 / 1024 rows 11.7 / 49.6 -> 11.4 / 46.7 us).
  RowInfo ri;
  f32x4_t co, si;
  if constexpr (MODE == F_QKV) {
    if (wave < MT) {
      const int rc = min(m0 + wave * 16 + r, M - 1);
      ri = fa.rows[rc];
      const float* c = fa.cs + (size_t)rc * fa.d_head + t0 + 4 * (kg & 1);
      co = *reinterpret_cast<const f32x4_t*>(c);
      si = *reinterpret_cast<const f32x4_t*>(c + half);
    }
  }
  // Several short chains of additions per result instead of one long one, and their sums taken in 64 bits: the error
  // against 64-bit arithmetic stays below that of the plain kernel (64 lanes with a few terms each, added pairwise),
  // which float32 sums of the chains miss by 2 % (the matrix unit rounds inside its four-term step).
  constexpr int CH = MT == 1 ? 8 : 4;
  f32x4_t acc[CH][NS][MT], sq[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) sq[mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int a = 0; a < NS; ++a)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[c][a][mt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  for (int s0 = s_begin; s0 < s_end; s0 += F_D) {
    f32x4_t wf[F_D][NS], xf[F_D][MT], gn[NORM ? F_D : 1];
#pragma unroll
    for (int j = 0; j < F_D; ++j) {
      const int p = (s0 + j) * 4 + kg;
      const bool in = s0 + j < s_end && p < pieces;          // k past the end multiplies as zero
      const int pc = in ? p : 0;
#pragma unroll
      for (int a = 0; a < NS; ++a) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(w[a] + pc * 4);
        wf[j][a] = in ? v : (f32x4_t){0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(x[mt] + pc * 4);
        xf[j][mt] = in ? v : (f32x4_t){0.f, 0.f, 0.f, 0.f};
      }
      if constexpr (NORM) gn[j] = *reinterpret_cast<const f32x4_t*>(fa.gain + pc * 4);
    }
    if constexpr (NORM) {
#pragma unroll
      for (int j = 0; j < F_D; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          sq[mt] += xf[j][mt] * xf[j][mt];
          xf[j][mt] *= gn[j];
        }
    }
#pragma unroll
    for (int j = 0; j < F_D; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int a = 0; a < NS; ++a)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[(j * 4 + i) % CH][a][mt] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(wf[j][a][i], xf[j][mt][i], acc[(j * 4 + i) % CH][a][mt], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < NS; ++a)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      f32x4_t t;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        double d = 0.0;
#pragma unroll
        for (int c = 0; c < CH; ++c) d += (double)acc[c][a][mt][i];
        t[i] = (float)d;
      }
      s_acc[wave][a * MT + mt][lane] = t;
    }
  if constexpr (NORM) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      double t = ((double)sq[mt][0] + (double)sq[mt][1]) + ((double)sq[mt][2] + (double)sq[mt][3]);
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      if (lane < 16) s_ss[wave][mt][lane] = t;
    }
  }
  __syncthreads();
  if (wave >= MT) return;
  // wave mt finishes row tile mt: row r, columns n0 + 4 * kg .. + 3
  double y[NS][4];
#pragma unroll
  for (int a = 0; a < NS; ++a) {
    f32x4_t p[F_WAVES];
#pragma unroll
    for (int v = 0; v < F_WAVES; ++v) p[v] = s_acc[v][a * MT + wave][lane];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double d = 0.0;
#pragma unroll
      for (int v = 0; v < F_WAVES; ++v) d += (double)p[v][i];
      y[a][i] = d;
    }
  }
  if constexpr (NORM) {
    double t = 0.0;
#pragma unroll
    for (int v = 0; v < F_WAVES; ++v) t += s_ss[v][wave][r];
    const double scale = 1.0 / sqrt(t / (double)K + (double)fa.eps);
#pragma unroll
    for (int a = 0; a < NS; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i) y[a][i] *= scale;
  }
  const int m = m0 + wave * 16 + r, n = n0 + 4 * kg;
  f32x4_t o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = (float)y[0][i];
  if constexpr (MODE == F_QKV) {
    f32x4_t b;
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = __shfl_xor(o[i], 32, 64);
    if (m >= M) return;
    const int t = t0 + 4 * (kg & 1), col = t + (kg >> 1) * half;
    if (head < fa.n_q + fa.n_kv) o = kg < 2 ? o * co - b * si : o * co + b * si;
    float* dst = out + ((size_t)m * fa.n_q + head) * fa.d_head;
    if (head >= fa.n_q) {
      const int value = head >= fa.n_q + fa.n_kv, kvh = head - fa.n_q - value * fa.n_kv;
      dst = reinterpret_cast<float*>(fa.g.kv + ((size_t)(fa.layer * 2 + value) * fa.n_kv + kvh) * fa.g.plane_bytes +
                                     (size_t)sp_phys_slot(fa.g, ri.req, ri.base, ri.P + ri.node) * fa.g.row_bytes);
    }
    *reinterpret_cast<f32x4_t*>(dst + col) = o;
    return;
  }
  if (m >= M) return;
  if (GATEUP) {
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = o[i] / (1.f + __expf(-o[i])) * (float)y[NS - 1][i];
  }
  const float* h = out + (size_t)m * N + n;
  float* dst = (MODE == F_OUT ? reinterpret_cast<float*>(fa.plan->x_out) : out) + (size_t)m * N + n;
  constexpr bool ADD = MODE == F_RESIDUAL || MODE == F_OUT;
  if (n + 4 <= N && (N & 3) == 0) {
    if (ADD) {
      const f32x4_t hv = *reinterpret_cast<const f32x4_t*>(h);
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (float)((double)hv[i] + y[0][i]);
    }
    *reinterpret_cast<f32x4_t*>(dst) = o;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) if (n + i < N) dst[i] = ADD ? (float)((double)h[i] + y[0][i]) : o[i];
  }
}

// Tree attention, one workgroup per (row, query head): every wave takes a quarter of the visible range, 64 slots at a
// time -- scores with a slot per lane, then the weighted sum of the V rows with the head's columns across the lanes --
// and keeps an online softmax; the four states are folded at the end.
template <int DH>
__global__ void __launch_bounds__(256) k_attn_f32(const float* __restrict__ q, const RowInfo* rows, const ReqTables* tables,
                                                  KvGeom g, int layer, float* __restrict__ out, int n_q, int n_kv) {
  constexpr int C = DH / 64;               // columns per lane
  __shared__ __attribute__((aligned(16))) float s_q[DH];
  __shared__ __attribute__((aligned(16))) float s_p[4][64];
  __shared__ int s_slot[4][64];
  __shared__ float s_o[4][DH], s_m[4], s_l[4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int row = blockIdx.x / n_q, head = blockIdx.x - row * n_q;
  const int kvh = head / (n_q / n_kv);
  if ((int)threadIdx.x < DH) s_q[threadIdx.x] = q[((size_t)row * n_q + head) * DH + threadIdx.x];
  const RowInfo ri = rows[row];
  unsigned long long anc[SP_W];
#pragma unroll
  for (int w = 0; w < SP_W; ++w) anc[w] = tables[ri.req].anc[ri.node][w];
  const float* kplane = reinterpret_cast<const float*>(g.kv + ((size_t)(layer * 2 + 0) * n_kv + kvh) * g.plane_bytes);
  const float* vplane = reinterpret_cast<const float*>(g.kv + ((size_t)(layer * 2 + 1) * n_kv + kvh) * g.plane_bytes);
  const float scale = rsqrtf((float)DH);
  const int total = ri.P + ri.T;
  const int c0 = (int)((long long)total * wave / 4), c1 = (int)((long long)total * (wave + 1) / 4);
  float mx = -INFINITY, l = 0.f, o[8][C];      // eight chains of additions per column
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int c = 0; c < C; ++c) o[e][c] = 0.f;
  __syncthreads();
  for (int s0 = c0; s0 < c1; s0 += 64) {
    const int s = s0 + lane;
    const bool in = s < c1;
    bool vis = in;
    if (in && s >= ri.P) {
      const int j = s - ri.P;
      unsigned long long word = 0ull;
#pragma unroll
      for (int w = 0; w < SP_W; ++w) word = (j >> 6) == w ? anc[w] : word;
      vis = (word >> (j & 63)) & 1ull;
    }
    // slots that are not visible read K of the request's first slot, which then does not count, and add nothing below
    const int slot = (int)sp_phys_slot(g, ri.req, ri.base, vis ? s : 0);
    const f32x4_t* k = reinterpret_cast<const f32x4_t*>(kplane + (size_t)slot * DH);
    f32x4_t d4 = {0.f, 0.f, 0.f, 0.f}, d4b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < DH / 4; t += 2) {
      d4 += k[t] * *reinterpret_cast<const f32x4_t*>(&s_q[t * 4]);
      d4b += k[t + 1] * *reinterpret_cast<const f32x4_t*>(&s_q[t * 4 + 4]);
    }
    d4 += d4b;
    const float sc = vis ? ((d4[0] + d4[1]) + (d4[2] + d4[3])) * scale : -INFINITY;
    const float mn = fmaxf(mx, wave_max(sc));
    const float corr = mn == -INFINITY ? 1.f : __expf(mx - mn);          // 0 from -inf
    const float p = vis ? __expf(sc - mn) : 0.f;
    l = l * corr + wave_sum(p);
    mx = mn;
    s_p[wave][lane] = p;
    s_slot[wave][lane] = vis ? slot : -1;
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int c = 0; c < C; ++c) o[e][c] *= corr;
    __builtin_amdgcn_wave_barrier();
    const int ns = min(64, c1 - s0);
    // sixteen V rows; where some are not visible these become zeros (a weight of zero would make NaN of an infinity)
    auto add16 = [&](int j, auto all_visible) {
      float pv[16], vv[16][C];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        pv[u] = s_p[wave][j + u];
        const int sl = s_slot[wave][j + u];
        const float* vp = vplane + (size_t)(all_visible.value ? sl : max(sl, 0)) * DH + lane;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const float v = vp[c * 64];
          vv[u][c] = all_visible.value || sl >= 0 ? v : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) o[u & 7][c] += pv[u] * vv[u][c];
    };
    int j = 0;
    for (const int lim = min(c1, ri.P) - s0; j + 16 <= min(ns, lim); j += 16) add16(j, std::true_type{});    // committed context
    for (; j < ns; j += 16) add16(j, std::false_type{});
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    s_o[wave][c * 64 + lane] = ((o[0][c] + o[1][c]) + (o[2][c] + o[3][c])) + ((o[4][c] + o[5][c]) + (o[6][c] + o[7][c]));
  if (lane == 0) { s_m[wave] = mx; s_l[wave] = l; }
  __syncthreads();
  if ((int)threadIdx.x >= DH) return;
  const float gm = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
  float num = 0.f, den = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float f = s_m[w] == -INFINITY ? 0.f : __expf(s_m[w] - gm);
    num += s_o[w][threadIdx.x] * f;
    den += s_l[w] * f;
  }
  out[((size_t)row * n_q + head) * DH + threadIdx.x] = num / den;
}

template <int MODE>
static hipError_t launch_gemm_f32(const float* X, const float* W, float* out, int M, int N, int K, const F32Args& fa,
                                  hipStream_t st) {
  if (M < 1 || N < 1 || K < 4 || K % 4) return hipErrorInvalidValue;
  const int tiles = (M + 15) / 16, mt = tiles >= 4 ? 4 : tiles >= 2 ? 2 : 1;     // row tiles that share a read of the weights
  const dim3 grid((N + 15) / 16, (tiles + mt - 1) / mt);
#define SP_GO(MTV) hipLaunchKernelGGL((k_gemm_f32<MTV, MODE>), grid, dim3(64 * F_WAVES), 0, st, X, W, out, M, N, K, fa)
  if (mt == 1) SP_GO(1); else if (mt == 2) SP_GO(2); else SP_GO(4);
#undef SP_GO
  return hipGetLastError();
}
hipError_t sp_launch_gemm_f32(const float* X, const float* W, float* out, int M, int N, int K, hipStream_t st) {
  return launch_gemm_f32<F_PLAIN>(X, W, out, M, N, K, F32Args{}, st);
}
// RMSNorm and rotation cost every workgroup of QKV some 2.2 us (each column tile forms the norm of its rows again), a norm and a
// rotation of their own about 10 us together: joined up to four rounds of workgroups over the CUs (d = 512, 3072 columns:
// QKV 512 rows 57.2 / 43.7 us, 1024 rows 109 / 82; two layers at 384 rows 309 / 304).
bool sp_qkv_f32_joined(int M, int N, int n_cu) { return (long long)((M + 63) / 64) * ((N + 15) / 16) <= 4ll * n_cu; }
hipError_t sp_launch_qkv_f32(const float* h, const float* gain, float eps, const float* W, const RowInfo* rows, const float* cs,
                             float* qbuf, KvGeom g, int layer, int M, int d, int n_q, int n_kv, int d_head, hipStream_t st) {
  if (d_head < 16 || d_head % 16) return hipErrorInvalidValue;      // eight pairs to a workgroup
  F32Args fa{};
  fa.gain = gain; fa.eps = eps; fa.rows = rows; fa.cs = cs; fa.g = g; fa.layer = layer;
  fa.n_q = n_q; fa.n_kv = n_kv; fa.d_head = d_head;
  return launch_gemm_f32<F_QKV>(h, W, qbuf, M, (n_q + 2 * n_kv) * d_head, d, fa, st);
}
hipError_t sp_launch_gateup_f32(const float* h, const float* gain, float eps, const float* W, float* act, int M, int F, int K,
                                hipStream_t st) {
  F32Args fa{};
  fa.gain = gain; fa.eps = eps;
  return launch_gemm_f32<F_GATEUP>(h, W, act, M, F, K, fa, st);
}
hipError_t sp_launch_residual_f32(const float* X, const float* W, float* h, const AttnPlan* plan_out, int M, int N, int K,
                                  hipStream_t st) {
  F32Args fa{};
  fa.plan = plan_out;
  return plan_out ? launch_gemm_f32<F_OUT>(X, W, h, M, N, K, fa, st) : launch_gemm_f32<F_RESIDUAL>(X, W, h, M, N, K, fa, st);
}

hipError_t sp_launch_attn_f32(const float* q, const RowInfo* rows, const ReqTables* tables, KvGeom g, int layer, float* out,
                              int M, int n_q, int n_kv, int d_head, hipStream_t st) {
  const dim3 grid(M * n_q);
  if (d_head == 64) hipLaunchKernelGGL(k_attn_f32<64>, grid, dim3(256), 0, st, q, rows, tables, g, layer, out, n_q, n_kv);
  else if (d_head == 128) hipLaunchKernelGGL(k_attn_f32<128>, grid, dim3(256), 0, st, q, rows, tables, g, layer, out, n_q, n_kv);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
