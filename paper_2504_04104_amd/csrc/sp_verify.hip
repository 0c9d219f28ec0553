// Lossy verification at the last stage (Sec. 3.4, "Lossless and Lossy Acceleration"):
//   (1) relaxed: of the root's children, the one whose token the large model finds most
//       probable -- some child is always verified, the pipeline never stalls;
//   (2) top-p:   children whose token lies in the large model's top-p set (tokens in descending
//       probability, the shortest prefix whose mass reaches p) are acceptable; the one with the
//       highest draft probability wins; none acceptable = a miss as in the lossless case.
// Equal probabilities are ordered by ascending token id, equal candidates by ascending node.
//
// Input: one row of logits per request (the root's output through the final norm and the
// vocabulary matrix).  A token t is in the top-p set iff the mass of the tokens in front of it,
//   before(t) = sum over { v : l_v > l_t  or  (l_v == l_t and v < t) } of softmax(l)_v,
// is below p.  k_lossy_slices cuts the vocabulary into slices, one workgroup each: slice maximum
// and its first index, sum of exp(l - slice max), and, one lane per candidate, the slice's share
// of before(token of the candidate).  k_lossy_decide rescales and adds the slices in a fixed
// order (so the result does not depend on timing) and decides.
#include "sp_launch.h"

#define SLICE 2048        // most tokens of a slice

template <typename T>
__global__ void __launch_bounds__(1024) k_row_norm(const T* __restrict__ x, const T* __restrict__ gain,
                                                    T* __restrict__ xn, int d, float eps, bool frag) {
  __shared__ float s_red[16];
  const int row = blockIdx.x;
  const T* xr = x + (size_t)row * d;
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 1024) { const float v = Elt<T>::ld(xr + c); ss += v * v; }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) tot += s_red[w];
  const float rs = rsqrtf(tot / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += 1024)
    Elt<T>::st(xn + row_at(frag, row, c, d), Elt<T>::ld(xr + c) * rs * Elt<T>::ld(gain + c));
}

// The root's children in node order: s_node[0..nc), their tokens in s_tok.  Called by all threads (256 or more).
__device__ __forceinline__ int root_children(const ReqTables& t, int T, int* s_node, int* s_tok, int* s_wcount) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const bool is = tid < T && t.parent[tid] == -1;
  const unsigned long long bal = __ballot(is);
  if (lane == 0 && wave < 4) s_wcount[wave] = __popcll(bal);
  __syncthreads();
  int before = 0;
  for (int w = 0; w < min(wave, 4); ++w) before += s_wcount[w];
  if (is) {
    const int pos = before + __popcll(bal & ((1ull << lane) - 1ull));
    s_node[pos] = tid;
    s_tok[pos] = t.token[tid];
  }
  const int nc = s_wcount[0] + s_wcount[1] + s_wcount[2] + s_wcount[3];
  __syncthreads();
  return nc;
}

// A request's logits in memory: its row of [n][V], or of tiles of 1 << shift columns, [tile][n][column].
struct LogitRow {
  const float* row;
  int shift;
  size_t step;               // from one of its tiles to the next
  __device__ __forceinline__ LogitRow(const float* logits, int item, int n, int V, int tile_cols) {
    shift = tile_cols ? 31 - __clz(tile_cols) : 30;
    row = logits + (size_t)item * (tile_cols ? tile_cols : V);
    step = (size_t)n * (unsigned)tile_cols;
  }
  // (columns of a tile follow each other)
  __device__ __forceinline__ const float* at(int v) const { return row + (size_t)(v >> shift) * step + (v & ((1 << shift) - 1)); }
  __device__ __forceinline__ float operator[](int v) const { return *at(v); }
};

struct LossyBatch {
  int n, mode, V, slice, n_slices;
  int lie;                   // columns of the tiles that the logits lie in, or 0
  float top_p;
  int req[SP_BATCH];
};

// stats[item][slice] = (slice max, sum of exp(l - max), first index of the max as int bits, 0);
// before[item][slice][j] = sum over the slice's tokens in front of candidate j's token of exp(l - slice max).
__global__ void __launch_bounds__(256) k_lossy_slices(const ReqMeta* meta, const ReqTables* tables,
                                                       const float* __restrict__ logits, LossyBatch b, float* stats,
                                                       float* before) {
  __shared__ __attribute__((aligned(16))) float s_l[SLICE];
  __shared__ __attribute__((aligned(16))) float s_e[SLICE + 256];   // + the partial sums of the candidate pass
  __shared__ int s_node[SP_T], s_tok[SP_T], s_wcount[4];
  __shared__ float s_rv[4];
  __shared__ int s_ri[4];
  const int item = blockIdx.y, slice = blockIdx.x;
  const int req = b.req[item];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const LogitRow L(logits, item, b.n, b.V, b.lie);
  const int v0 = slice * b.slice, len = min(b.slice, b.V - v0);
  const int nc = root_children(tables[req], meta[req].T, s_node, s_tok, s_wcount);

  float bv = -INFINITY;
  int bi = 0x7fffffff;
  {
    float lv[SLICE / 256];                             // all loads first: one memory round trip, not eight
#pragma unroll
    for (int u = 0; u < SLICE / 256; ++u) lv[u] = (tid + u * 256 < len) ? L[v0 + tid + u * 256] : -INFINITY;
#pragma unroll
    for (int u = 0; u < SLICE / 256; ++u) {
      const int i = tid + u * 256;
      if (i < len) {
        s_l[i] = lv[u];
        if (lv[u] > bv) { bv = lv[u]; bi = v0 + i; }   // ascending i: the first of equal maxima stays
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(bv, off, 64);
    const int oi = __shfl_xor(bi, off, 64);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (lane == 0) { s_rv[wave] = bv; s_ri[wave] = bi; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w)
    if (s_rv[w] > bv || (s_rv[w] == bv && s_ri[w] < bi)) { bv = s_rv[w]; bi = s_ri[w]; }
  __syncthreads();
  const float ref = bv == -INFINITY ? 0.f : bv;        // a slice without a finite logit (masked padding rows) has no mass
  float z = 0.f;
  for (int i = tid; i < len; i += 256) {
    const float e = expf(s_l[i] - ref);
    s_e[i] = e;
    z += e;
  }
  z = wave_sum(z);
  if (lane == 0) s_rv[wave] = z;
  __syncthreads();
  if (tid == 0) {
    float* st = stats + ((size_t)item * b.n_slices + slice) * 4;
    st[0] = bv;
    st[1] = (s_rv[0] + s_rv[1]) + (s_rv[2] + s_rv[3]);
    reinterpret_cast<int*>(st)[2] = bi;
    st[3] = 0.f;
  }
  if (b.mode == 1) return;                             // the relaxed rule compares logits, not masses
  // Candidate against every token of the slice: `width` threads side by side are candidates (a power of two, 16 at least), and
  // the 256 / width parts of the workgroup take their share of the slice each.  All threads of a part read the same LDS words (a
  // broadcast), four tokens per read.  The parts are added in order afterwards, so the sum does not depend on timing.  This
  // pass bounds the kernel where there are many requests (14 of 27 candidates each over 128256 tokens 52.7 -> 27.0 us, 28 of 17
  // whole calls 305 -> 262; before, a candidate took a lane of a whole wave and every token was looked at for a tie).
  __syncthreads();
  int width = 16;
  while (width < nc) width *= 2;
  const int parts = 256 / width, cand = tid & (width - 1), part = tid / width;
  float* s_part = s_e + SLICE;                       // [256] partial sums, behind the exponentials
  {
    float acc = 0.f;
    const int tk = cand < nc ? s_tok[cand] : -1;
    const bool valid = tk >= 0 && tk < b.V;
    const float thr = valid ? L[tk] : INFINITY;
    const int rel = tk - v0;                         // tokens of the slice with index < rel come first among equals
    const int per = ((len + parts - 1) / parts + 3) & ~3;
    const int i0 = min(part * per, len), i1 = min(i0 + per, len);
    // a part in front of the candidate's token counts the equal ones too: those above the next float below (equal masked
    // tokens have no mass, and nothing is above a threshold that is no number)
    const float bar = rel < i1 || thr == -INFINITY ? thr : nextafterf(thr, -INFINITY);
    if (__builtin_amdgcn_ballot_w64(valid && rel >= i0 && rel < i1) == 0) {
      int i = i0;
      for (; i + 4 <= i1; i += 4) {
        const f32x4_t l4 = *reinterpret_cast<const f32x4_t*>(&s_l[i]);
        const f32x4_t e4 = *reinterpret_cast<const f32x4_t*>(&s_e[i]);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += l4[u] > bar ? e4[u] : 0.f;
      }
      for (; i < i1; ++i) acc += s_l[i] > bar ? s_e[i] : 0.f;
    } else {
      int i = i0;
      for (; i + 4 <= i1; i += 4) {
        const f32x4_t l4 = *reinterpret_cast<const f32x4_t*>(&s_l[i]);
        const f32x4_t e4 = *reinterpret_cast<const f32x4_t*>(&s_e[i]);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += (l4[u] > thr || (l4[u] == thr && i + u < rel)) ? e4[u] : 0.f;
      }
      for (; i < i1; ++i) acc += (s_l[i] > thr || (s_l[i] == thr && i < rel)) ? s_e[i] : 0.f;
    }
    s_part[tid] = valid ? acc : 0.f;
  }
  __syncthreads();
  if (tid < nc) {
    float acc = 0.f;
    for (int q = 0; q < parts; ++q) acc += s_part[q * width + tid];
    before[((size_t)item * b.n_slices + slice) * SP_T + tid] = acc;
  }
}

// out[2*item] = verified node or -1, out[2*item+1] = the model's top-1 token, which also becomes the
// root's stored prediction (what a miss falls back to).  A chain of latencies: every step over slices or
// candidates is taken by all sixteen waves (one request, 64 candidates: 15.7 us with 63 slices before, 13.1 us with 251).
__global__ void __launch_bounds__(1024) k_lossy_decide(ReqMeta* meta, const ReqTables* tables,
                                                        const float* __restrict__ logits, LossyBatch b,
                                                        const float* stats, const float* before, int* out) {
  constexpr int BLK = 1024;              // slices per round
  __shared__ int s_node[SP_T], s_tok[SP_T], s_wcount[4];
  __shared__ float s_sc[BLK], s_part[16][64], s_red[16], s_before[SP_T];
  __shared__ int s_redi[16];
  const int item = blockIdx.x, req = b.req[item], tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const ReqTables& t = tables[req];
  const LogitRow L(logits, item, b.n, b.V, b.lie);
  const float* st = stats + (size_t)item * b.n_slices * 4;
  // the slices' maxima are asked for before the walk over the tables
  float m = -INFINITY;
  int top1 = 0x7fffffff;
  for (int q = tid; q < b.n_slices; q += 1024) {
    const float v = st[q * 4];
    const int i = reinterpret_cast<const int*>(st)[q * 4 + 2];
    if (v > m || (v == m && i < top1)) { m = v; top1 = i; }
  }
  const int nc = root_children(t, meta[req].T, s_node, s_tok, s_wcount);
  // larger value first, the lower index among equal ones; the same answer in every thread
  auto block_top = [&](float& v, int& i) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const float ov = __shfl_xor(v, off, 64);
      const int oi = __shfl_xor(i, off, 64);
      if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
    }
    __syncthreads();
    if (lane == 0) { s_red[wave] = v; s_redi[wave] = i; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 16; ++w)
      if (s_red[w] > v || (s_red[w] == v && s_redi[w] < i)) { v = s_red[w]; i = s_redi[w]; }
  };
  // what the candidates are ranked by: the token's logit (relaxed) or its draft probability
  float Z = 0.f;
  const bool mine = tid < nc;
  const int tk = mine ? s_tok[tid] : -1;
  const bool valid = tk >= 0 && tk < b.V;
  const float key = !valid ? -INFINITY : b.mode == 1 ? L[tk] : t.prob[s_node[tid]];
  block_top(m, top1);

  if (b.mode == 2) {
    // waves as candidate groups of 64 times runs of slices; a run's slices are read eight at a time
    const int groups = (nc + 63) >> 6, runs = groups > 0 ? 16 / groups : 1;
    const int cg = groups > 0 ? wave % groups : 0, run = groups > 0 ? wave / groups : runs;
    float z = 0.f, acc = 0.f;
    for (int q0 = 0; q0 < b.n_slices; q0 += BLK) {
      const int ns = min(BLK, b.n_slices - q0);
      __syncthreads();
      if (tid < ns) {
        const float top = st[(q0 + tid) * 4];
        const float sc = top == -INFINITY ? 0.f : expf(top - m);   // (m may be minus infinity itself)
        s_sc[tid] = sc;
        z += st[(q0 + tid) * 4 + 1] * sc;
      }
      __syncthreads();
      if (run < runs) {
        const float* bp = before + ((size_t)item * b.n_slices + q0) * SP_T + cg * 64 + lane;
        const bool in = cg * 64 + lane < nc;
        const int a0 = ns * run / runs, a1 = ns * (run + 1) / runs;
        int q = a0;
        for (; q + 8 <= a1; q += 8) {
          float v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = in ? bp[(size_t)(q + u) * SP_T] : 0.f;
#pragma unroll
          for (int u = 0; u < 8; ++u) acc += v[u] * s_sc[q + u];
        }
        for (; q < a1; ++q) acc += (in ? bp[(size_t)q * SP_T] : 0.f) * s_sc[q];
      }
    }
    z = wave_sum(z);
    __syncthreads();
    if (lane == 0) s_red[wave] = z;
    s_part[wave][lane] = acc;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 16; ++w) Z += s_red[w];
    if (mine) {
      float bf = 0.f;
      for (int q = 0; q < runs; ++q) bf += s_part[q * groups + (tid >> 6)][tid & 63];
      s_before[tid] = bf;
    }
  }
  const bool ok = valid && (b.mode == 1 || s_before[tid] < b.top_p * Z);
  // the first acceptable candidate stays if its key is no number; other keys that are none never win
  float first_key = 0.f;
  int first = ok ? tid : 0x7fffffff;
  {
    float minus = ok ? -(float)tid : -INFINITY;
    block_top(minus, first);
    __syncthreads();
    if (tid == first) s_red[0] = key;
    __syncthreads();
    first_key = first != 0x7fffffff ? s_red[0] : 0.f;
    __syncthreads();
  }
  float bk = ok && key == key ? key : -INFINITY;
  int best = ok && key == key ? tid : 0x7fffffff;
  block_top(bk, best);
  if (tid == 0) {
    if (first != 0x7fffffff && first_key != first_key) best = first;
    out[2 * item] = best == 0x7fffffff ? -1 : s_node[best];
    out[2 * item + 1] = top1;
    meta[req].root_pred = top1;
  }
}

// ---------------------------------------------------------------------------------------------
// Stochastic verification (Sec. 4.3, "Stochastic Decoding"): the token after the root is drawn from
// the large model's distribution at temperature T, among the candidates collected in descending
// probability until their probabilities sum to top_p or top_k of them have been taken (equal
// probabilities by ascending token id); the draw is the inverse CDF of the candidates' renormalised
// probabilities at a uniform number the caller supplies.  The drawn token takes the place of the
// top-1 token: it becomes the root's prediction, and the verified node is the first root child that
// carries it (-1: a stall).
// One workgroup of 1024 threads per request: row maximum, normaliser over the whole vocabulary, the
// top_k-th largest logit by a radix select over the order-preserving bit pattern (four passes of 8
// bits, one histogram per wave), an index-ordered gather of the logits above it and of the first
// ones equal to it, a sort by counting, and the running sums by one wave.
struct SampleBatch {
  int n, V, top_k;
  int lie;                   // columns of the tiles that the logits lie in, or 0
  int tile_cols;             // STATS: columns per statistics entry
  const float* stats;        // STATS: [n][V / tile_cols] pairs (maximum, sum of exp((l - maximum) / T))
  float inv_T, top_p;
  int req[SP_BATCH];
  float u[SP_BATCH];
};

__device__ __forceinline__ uint32_t order_key(float f) {           // ascending like the floats themselves
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__device__ __forceinline__ unsigned long long sample_key(float l, int idx) {
  return (unsigned long long)order_key(l) << 32 | (unsigned long long)(0xffffffffu - (unsigned)idx);
}

// Eight loads of W floats per thread, all issued before the first use: one workgroup reads the whole row, so
// with a load per iteration a pass would be a chain of V / 1024 memory latencies.  W = 4 needs V % 4 == 0
// (then an index below V is followed by three more).  Index of element (u, c): base + (u * 1024 + tid) * W + c.
template <int W>
__device__ __forceinline__ void sample_load(const LogitRow& L, int V, int base, int tid, float (&v)[8][W]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int i = base + (u * 1024 + tid) * W;
    if constexpr (W == 4) {
      const float4 t = i < V ? *reinterpret_cast<const float4*>(L.at(i)) : make_float4(0.f, 0.f, 0.f, 0.f);
      v[u][0] = t.x; v[u][1] = t.y; v[u][2] = t.z; v[u][3] = t.w;
    } else {
      v[u][0] = i < V ? L[i] : 0.f;
    }
  }
}

#define SP_SAMPLE_CAND 2048   // candidates the short path can hold

// One workgroup per request.  The K = top_k largest logits are found without ordering the row: every thread
// keeps the maximum of the elements it reads, a wave takes the ceil(K / 16) largest of its 64 thread maxima,
// and the smallest of those 16 * ceil(K / 16) >= K distinct elements is a lower bound t0 of the K-th largest
// logit.  A second pass collects the elements >= t0 (a few hundred on a spread-out row) and their places follow
// from counting.  Rows that defeat the bound (long runs of equal logits, vocabularies under a few thousand)
// take a radix selection over the whole row instead.
// STATS: the kernel that formed the logits left every tile's maximum and exponential sum.  The tile maxima take the
// place of the thread maxima, the normaliser is added up from the tiles, and only the tiles whose maximum reaches the
// bound (some K of a thousand) are read: one workgroup no longer walks the row twice (32 requests over 128256 tokens:
// 53 -> 15 us).
template <int W, bool STATS>
__global__ void __launch_bounds__(1024) k_sample_decide(ReqMeta* meta, const ReqTables* tables,
                                                         const float* __restrict__ logits, SampleBatch b, int* out) {
  __shared__ float s_f[16], s_g[16];
  __shared__ unsigned s_hist[16][256];
  __shared__ unsigned s_scan[16];
  __shared__ unsigned s_pick[2];                  // digit chosen by a pass, and how many of the top_k are still to find below it
  __shared__ uint32_t s_key[SP_SAMPLE_MAX_K], s_skey[SP_SAMPLE_MAX_K];
  __shared__ int s_idx[SP_SAMPLE_MAX_K], s_sidx[SP_SAMPLE_MAX_K];
  // the short path's candidates: key above the complemented index, so that a larger number comes first (distinct)
  __shared__ __attribute__((aligned(16))) unsigned long long s_cand[SP_SAMPLE_CAND + 8];
  __shared__ int s_rank[SP_SAMPLE_CAND];
  __shared__ unsigned s_ncand;
  __shared__ int s_tok, s_best;
  const int item = blockIdx.x, req = b.req[item];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const LogitRow L(logits, item, b.n, b.V, b.lie);
  const int V = b.V, K = min(b.top_k, V);

  // first pass: thread maxima, from them the row maximum and the bound t0
  float tm = -INFINITY;
  const int n_tiles = STATS ? V / b.tile_cols : 0;
  const float2* ts = reinterpret_cast<const float2*>(b.stats) + (size_t)item * n_tiles;
  if (STATS)
    for (int t = lane * 16 + wave; t < n_tiles; t += 1024) tm = fmaxf(tm, ts[t].x);   // every wave gets its share
  for (int base = 0; !STATS && base < V; base += 8 * 1024 * W) {
    float v[8][W];
    sample_load<W>(L, V, base, tid, v);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (base + (u * 1024 + tid) * W < V) {
#pragma unroll
        for (int c = 0; c < W; ++c) tm = fmaxf(tm, v[u][c]);
      }
  }
  {
    const float wmx = wave_max(tm);
    float cur = tm, kept = wmx;
    const int rounds = (K + 15) >> 4;
    for (int r = 0; r < rounds; ++r) {           // the wave's r-th largest thread maximum, one thread retired per round
      kept = wave_max(cur);
      const unsigned long long holders = __ballot(cur == kept);
      if (holders == 0ull) { kept = -INFINITY; break; }          // only NaNs left
      if (lane == (int)__builtin_ctzll(holders)) cur = -INFINITY;
    }
    if (lane == 0) { s_f[wave] = wmx; s_g[wave] = kept; }
    if (tid == 0) s_ncand = 0u;
  }
  __syncthreads();
  float mx = s_f[0], t0 = s_g[0];
#pragma unroll
  for (int w = 1; w < 16; ++w) { mx = fmaxf(mx, s_f[w]); t0 = fminf(t0, s_g[w]); }
  __syncthreads();

  // second pass: the normaliser of softmax(l / T) over the whole vocabulary, added in a fixed order, and the candidates
  float z = 0.f;
  if (STATS) {
    int* s_tile = reinterpret_cast<int*>(&s_hist[0][0]);          // the tiles to read; a longer list than this is cut ...
    constexpr int TILES_MAX = 16 * 256;
    if (tid == 0) s_pick[0] = 0u;
    __syncthreads();
    for (int t = tid; t < n_tiles; t += 1024) {
      const float2 p = ts[t];
      z += p.y * (p.x == mx || p.x == -INFINITY ? 1.f : expf((p.x - mx) * b.inv_T));
      if (p.x >= t0) {
        const unsigned at = atomicAdd(&s_pick[0], 1u);
        if (at < TILES_MAX) s_tile[at] = t;
      }
    }
    __syncthreads();
    const int n_pick = (int)s_pick[0], cols = b.tile_cols;
    if (n_pick > TILES_MAX) {
      if (tid == 0) s_ncand = SP_SAMPLE_CAND + 1u;                // ... and the whole row is searched instead
    } else {
      // a tile is 64 or 128 columns; four of a wave's tiles in flight
      for (int k0 = wave; k0 < n_pick; k0 += 64) {
        float2 v[4];
        int base[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k0 + u * 16;
          base[u] = k < n_pick ? s_tile[k] * cols : -1;
          v[u] = make_float2(-INFINITY, -INFINITY);
          if (base[u] >= 0 && 2 * lane < cols) v[u] = *reinterpret_cast<const float2*>(L.at(base[u]) + 2 * lane);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (base[u] < 0 || 2 * lane >= cols) continue;
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const float l = c == 0 ? v[u].x : v[u].y;
            if (l >= t0) {
              const unsigned p = atomicAdd(&s_ncand, 1u);
              if (p < SP_SAMPLE_CAND) s_cand[p] = sample_key(l, base[u] + 2 * lane + c);
            }
          }
        }
      }
    }
  }
  for (int base = 0; !STATS && base < V; base += 8 * 1024 * W) {
    float v[8][W];
    sample_load<W>(L, V, base, tid, v);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = base + (u * 1024 + tid) * W;
      if (i < V) {
#pragma unroll
        for (int c = 0; c < W; ++c) {
          z += expf((v[u][c] - mx) * b.inv_T);
          if (v[u][c] >= t0) {
            const unsigned p = atomicAdd(&s_ncand, 1u);
            if (p < SP_SAMPLE_CAND) s_cand[p] = sample_key(v[u][c], i + c);
          }
        }
      }
    }
  }
  z = wave_sum(z);
  if (lane == 0) s_f[wave] = z;
  __syncthreads();
  float Z = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) Z += s_f[w];
  const int n_cand = (int)s_ncand;

  if (n_cand <= SP_SAMPLE_CAND) {
    // descending probability, equal ones by ascending token id: a candidate's place is the number that beat it,
    // counted by several threads per candidate, each over its run of the list, eight candidates per step
    int span = 64;                                   // candidates a pass of the threads covers
    while (span < n_cand && span < 1024) span <<= 1;
    const int parts = 1024 / span, part = tid / span;
    const int per = ((n_cand + parts - 1) / parts + 7) & ~7;
    const int j0 = min(part * per, n_cand), j1 = min(j0 + per, n_cand);
    for (int i = tid; i < n_cand; i += 1024) s_rank[i] = 0;
    if (tid < 8) s_cand[n_cand + tid] = 0ull;        // beats nobody
    __syncthreads();
    for (int i = tid % span; i < n_cand; i += span) {
      const unsigned long long k = s_cand[i];
      int rank = 0;
      for (int j = j0; j < j1; j += 8) {
        unsigned long long o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = s_cand[j + e];
#pragma unroll
        for (int e = 0; e < 8; ++e) rank += (o[e] > k && j + e < j1) ? 1 : 0;
      }
      if (parts == 1) s_rank[i] = rank;
      else atomicAdd(&s_rank[i], rank);
    }
    __syncthreads();
    for (int i = tid; i < n_cand; i += 1024)
      if (s_rank[i] < K) {
        const unsigned long long k = s_cand[i];
        s_skey[s_rank[i]] = (uint32_t)(k >> 32);
        s_sidx[s_rank[i]] = (int)(0xffffffffu - (unsigned)k);
      }
  } else {
    // the K-th largest key: fix its bytes from the top, counting the keys that share the bytes fixed so far
    uint32_t prefix = 0u, mask = 0u;
    unsigned need = (unsigned)K;
    for (int shift = 24; shift >= 0; shift -= 8) {
      for (int i = tid; i < 16 * 256; i += 1024) (&s_hist[0][0])[i] = 0u;
      __syncthreads();
      for (int base = 0; base < V; base += 8 * 1024 * W) {
        float v[8][W];
        sample_load<W>(L, V, base, tid, v);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (base + (u * 1024 + tid) * W < V) {
#pragma unroll
            for (int c = 0; c < W; ++c) {
              const uint32_t k = order_key(v[u][c]);
              if ((k & mask) == prefix) atomicAdd(&s_hist[wave][(k >> shift) & 255u], 1u);
            }
          }
        }
      }
      __syncthreads();
      if (tid < 256) {
        unsigned c = 0u;
#pragma unroll
        for (int w = 0; w < 16; ++w) c += s_hist[w][tid];
        s_hist[0][tid] = c;
      }
      __syncthreads();
      if (tid == 0) {
        unsigned above = 0u;
        int bin = 255;
        for (; bin > 0; --bin) {
          if (above + s_hist[0][bin] >= need) break;
          above += s_hist[0][bin];
        }
        s_pick[0] = (unsigned)bin;
        s_pick[1] = need - above;
      }
      __syncthreads();
      prefix |= s_pick[0] << shift;
      mask |= 255u << shift;
      need = s_pick[1];
      __syncthreads();
    }
    const uint32_t kth = prefix;                    // `need` of the keys equal to it belong to the top K: those with the lowest index
    const int n_gt = K - (int)need;

    // gather in index order: wave w owns the indices [w * seg, (w + 1) * seg) and reads them 64 at a time, so a
    // candidate's place is the count of the waves in front, of the rows in front and of the lower lanes of its row
    const int seg = (((V + 15) >> 4) + 63) & ~63;
    const int w0 = min(wave * seg, V), w1 = min(w0 + seg, V);
    unsigned c_gt = 0u, c_eq = 0u;                  // wave-uniform
    for (int r0 = w0; r0 < w1; r0 += 16 * 64) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) { const int i = r0 + u * 64 + lane; v[u] = i < w1 ? L[i] : 0.f; }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const bool in = r0 + u * 64 + lane < w1;
        const uint32_t k = order_key(v[u]);
        c_gt += (unsigned)__popcll(__ballot(in && k > kth));
        c_eq += (unsigned)__popcll(__ballot(in && k == kth));
      }
    }
    if (lane == 0) s_scan[wave] = (c_gt << 16) | min(c_eq, 0xffffu);   // more equal keys than that: only the first `need` matter
    __syncthreads();
    unsigned base = 0u;
    for (int w = 0; w < wave; ++w) {                 // saturating in the low half: the sum is only compared with `need`
      const unsigned sw = s_scan[w];
      base = ((base >> 16) + (sw >> 16)) << 16 | min((base & 0xffffu) + (sw & 0xffffu), 0xffffu);
    }
    int p_gt = (int)(base >> 16), p_eq = (int)(base & 0xffffu);
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int r0 = w0; r0 < w1; r0 += 16 * 64) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) { const int i = r0 + u * 64 + lane; v[u] = i < w1 ? L[i] : 0.f; }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int i = r0 + u * 64 + lane;
        const bool in = i < w1;
        const uint32_t k = order_key(v[u]);
        const unsigned long long m_gt = __ballot(in && k > kth), m_eq = __ballot(in && k == kth);
        if (in && k > kth) { const int p = p_gt + __popcll(m_gt & below); s_key[p] = k; s_idx[p] = i; }
        if (in && k == kth) {
          const int p = p_eq + __popcll(m_eq & below);
          if (p < (int)need) { s_key[n_gt + p] = k; s_idx[n_gt + p] = i; }
        }
        p_gt += __popcll(m_gt);
        p_eq = min(p_eq + __popcll(m_eq), 0xffff);
      }
    }
    __syncthreads();
    if (tid < K) {
      const uint32_t k = s_key[tid];
      const int ix = s_idx[tid];
      int rank = 0;
      for (int j = 0; j < K; ++j) rank += (s_key[j] > k) || (s_key[j] == k && s_idx[j] < ix);
      s_skey[rank] = k;
      s_sidx[rank] = ix;
    }
  }
  if (tid == 0) s_best = 0x7fffffff;
  __syncthreads();
  // running sums until top_p is reached (or the K candidates are used up), then the inverse CDF at u: one wave, two
  // candidates per lane (SP_SAMPLE_MAX_K = 128)
  if (wave == 0) {
    static_assert(SP_SAMPLE_MAX_K <= 128, "two candidates per lane");
    float p[2], run[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int j = 2 * lane + e;
      p[e] = j < K ? expf((key_value(s_skey[j]) - mx) * b.inv_T) / Z : 0.f;
    }
    // added one by one in candidate order: sums that never fall, and no candidate of probability zero with an interval
    // of its own (a scan in tree order differs by a rounding from lane to lane, and u near one drew such candidates)
    float sum = 0.f;
    run[0] = run[1] = 0.f;
    for (int j0 = 0; 2 * j0 < K; j0 += 8) {           // (probabilities past the K-th are zero)
      float a[8], c[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        a[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(p[0]), j0 + j));
        c[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(p[1]), j0 + j));
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float r0 = sum + a[j];
        sum = r0 + c[j];
        if (lane == j0 + j) { run[0] = r0; run[1] = sum; }
      }
    }
    // m candidates: up to and including the first whose running sum reaches top_p
    int m = K;
#pragma unroll
    for (int e = 1; e >= 0; --e) {
      const unsigned long long hit = __ballot(2 * lane + e < K && run[e] >= b.top_p);
      if (hit) m = min(m, 2 * (int)__builtin_ctzll(hit) + e + 1);
    }
    const float total = __shfl(((m - 1) & 1) ? run[1] : run[0], (m - 1) >> 1, 64);
    const float x = b.u[item] * total;
    int pick = m - 1;
#pragma unroll
    for (int e = 1; e >= 0; --e) {
      const unsigned long long hit = __ballot(2 * lane + e < m && x < run[e]);
      if (hit) pick = min(pick, 2 * (int)__builtin_ctzll(hit) + e);
    }
    if (lane == 0) s_tok = s_sidx[pick];
  }
  __syncthreads();
  const int tok = s_tok;
  const ReqTables& t = tables[req];
  if (tid < meta[req].T && t.parent[tid] == -1 && t.token[tid] == tok) atomicMin(&s_best, tid);
  __syncthreads();
  if (tid == 0) {
    out[2 * item] = s_best == 0x7fffffff ? -1 : s_best;
    out[2 * item + 1] = tok;
    meta[req].root_pred = tok;
  }
}

hipError_t sp_launch_verify_sample(ReqMeta* meta, const ReqTables* tables, const float* logits, int n, const int* reqs,
                                   int V, float temperature, float top_p, int top_k, const float* u,
                                   const float* stats, int tile_cols, int* out, hipStream_t st) {
  SampleBatch b;
  b.n = n; b.V = V; b.top_k = top_k; b.lie = logits_lie(tile_cols); b.tile_cols = tile_cols; b.stats = stats; b.inv_T = 1.f / temperature; b.top_p = top_p;
  for (int i = 0; i < n; ++i) { b.req[i] = reqs[i]; b.u[i] = u[i]; }
  // the bound needs ceil(top_k / 16) tiles for each of the 16 waves
  const bool tiles = stats && V / tile_cols >= 16 * ((top_k + 15) / 16);
  if (tiles)                                         // V % 64 == 0 there
    hipLaunchKernelGGL((k_sample_decide<4, true>), dim3(n), dim3(1024), 0, st, meta, tables, logits, b, out);
  else if (V % 4 == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0)
    hipLaunchKernelGGL((k_sample_decide<4, false>), dim3(n), dim3(1024), 0, st, meta, tables, logits, b, out);
  else
    hipLaunchKernelGGL((k_sample_decide<1, false>), dim3(n), dim3(1024), 0, st, meta, tables, logits, b, out);
  return hipGetLastError();
}

hipError_t sp_launch_row_norm(int dtype, const void* x, const void* gain, void* xn, bool frag, int M, int d, float eps,
                              hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(k_row_norm<float>, dim3(M), dim3(1024), 0, st, (const float*)x, (const float*)gain, (float*)xn, d, eps, false);
  else
    hipLaunchKernelGGL(k_row_norm<bf16_t>, dim3(M), dim3(1024), 0, st, (const bf16_t*)x, (const bf16_t*)gain, (bf16_t*)xn, d, eps, frag);
  return hipGetLastError();
}

// Tokens per slice: short slices where few requests would leave most of the chip idle (one request over 128256 tokens:
// 63 workgroups of 2048 tokens 37 us, 251 of 512 tokens 13 us), 2048 where the batch or the scratch memory asks for it.
static int lossy_slice(int n, int V, size_t scratch_floats) {
  for (int slice = 512; slice < SLICE; slice *= 2) {
    const size_t slices = (size_t)(V + slice - 1) / slice;
    if ((size_t)n * slices <= 512 && (size_t)n * slices * (4 + SP_T) <= scratch_floats) return slice;
  }
  return SLICE;
}

size_t sp_lossy_scratch_floats(int n, int V) {
  const size_t slices = (size_t)(V + SLICE - 1) / SLICE;
  return (size_t)n * slices * (4 + SP_T);
}

hipError_t sp_launch_verify_lossy(ReqMeta* meta, const ReqTables* tables, const float* logits, int tile_cols, int n, const int* reqs,
                                  int V, int mode, float top_p, float* scratch, size_t scratch_floats, int* out, hipStream_t st) {
  LossyBatch b;
  b.n = n; b.mode = mode; b.V = V; b.lie = logits_lie(tile_cols); b.slice = lossy_slice(n, V, scratch_floats);
  b.n_slices = (V + b.slice - 1) / b.slice; b.top_p = top_p;
  for (int i = 0; i < n; ++i) b.req[i] = reqs[i];
  float* stats = scratch;
  float* before = scratch + (size_t)n * b.n_slices * 4;
  hipLaunchKernelGGL(k_lossy_slices, dim3(b.n_slices, n), dim3(256), 0, st, meta, tables, logits, b, stats, before);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lossy_decide, dim3(n), dim3(1024), 0, st, meta, tables, logits, b, stats, before, out);
  return hipGetLastError();
}
