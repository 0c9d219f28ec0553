// Shared device-side definitions of the SpecPipe stage library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sp_plan.h"

#define SP_T 256          // tree capacity per request (== SP_MAX_TREE_NODES)
#define SP_W 4            // 64-bit words per ancestor-bitmask row

typedef uint16_t bf16_t;  // raw bfloat16 bits

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(8))) unsigned short u16x8_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;   // a 16-byte register quad

// ---- per-request device state -------------------------------------------------
// Counters of a request.  Written by the request-init, insert and prune kernels,
// read by the forward kernels; the host keeps a mirror only to validate arguments
// and to size launches.
struct ReqMeta {
  long long base;   // first cache slot of the request
  int cap;          // slots it owns
  int P;            // committed tokens (root included)
  int T;            // live speculative nodes
  int root_pred;    // the model's token after the committed context, -1 while unknown
};

// Tree tables of a request (Sec. 3.2: I, P, M) plus the map the last prune left
// for the cache compaction.  anc[i] holds row i of M as a bitmask: bit j set iff
// j == i or node j is an ancestor of node i.
struct ReqTables {
  int parent[SP_T];
  int depth[SP_T];
  int token[SP_T];
  float prob[SP_T];
  int pred[SP_T];         // the model's next token after the node, -1 until the last stage has seen it
  unsigned long long anc[SP_T][SP_W];
  // pending compaction: cache rows [0, n_kv_keep) of the tree region take the rows
  // of old nodes kv_src[0..n_kv_keep); rows below first_moved stay where they are.
  int pend_n_kv_keep;
  int pend_first_moved;
  int pend_P_old;
  int pend_T_old;
  short kv_src[SP_T];
  short tab_new[SP_T];    // old node -> new node index, -1 if it left the tables
};

// One row of a forward call.
struct RowInfo {
  long long base;   // request's first slot
  int req;
  int node;
  int pos;          // sequence position = P + depth
  int P;
  int T;
};

// A forward call's requests, passed to kernels by value.
struct FwdBatch {
  int n_req;
  int n_rows;
  int req[SP_BATCH];
  int first[SP_BATCH];
  int n[SP_BATCH];
  int row0[SP_BATCH];
};

// Arguments of one insert launch, passed by value: up to SP_T new nodes spread over up to
// SP_BATCH requests; request i owns entries [row0[i], row0[i+1]) and appends them after its
// t0[i] live nodes, in cache slots first_slot[i]...
// Paged cache: the pages that the requests take for these rows come along, in place of a launch per request that grows (32
// requests in steady state, pages of 64 slots: four of 4.5 us a pass, 843 -> 836 us): request i's logical pages pg_first[i] .. + pg_n[i] - 1 are page[pg_at[i]] and so on.
#define SP_INSERT_PAGES 32
struct InsertArgs {
  int n_req;
  short pg_first[SP_BATCH];
  unsigned char pg_n[SP_BATCH], pg_at[SP_BATCH];
  int page[SP_INSERT_PAGES];
  short req[SP_BATCH];
  short t0[SP_BATCH];
  short row0[SP_BATCH + 1];
  long long first_slot[SP_BATCH];   // base + prefix_len + t0 (logical slot prefix_len + t0 when paged)
  short parent[SP_T];
  int token[SP_T];
  float prob[SP_T];
};

struct PruneBatch {
  int n;
  int req[SP_BATCH];
  int mode[SP_BATCH];    // <0: skip
  int node[SP_BATCH];
};

#define SP_SAMPLE_MAX_K 128  // most candidates of a stochastic verification (== SP_MAX_SAMPLE_TOP_K)
#define SP_EXPAND_MAX 4096   // candidates of one fixed-width expansion (bottom tokens x k)

struct ExpandArgs {      // by value
  int req;
  int n_bottom;
  int k;
  int w;
  short bottom[SP_T];    // node whose children are proposed, ascending; -1 = the root (empty tree)
};

struct RowList {         // source rows of an in-place row compaction, by value
  int n_keep;
  int first_moved;
  short src[SP_T];
};

// ---- bf16 <-> f32 ---------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
// round-to-nearest-even in hardware (v_cvt_pk_bf16_f32)
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.f) & 0xffffu); }

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// Activations between the bf16 matrix-core kernels lie in fragment order: per 16 rows and 32 columns one block of 1 KB,
// lane-major as v_mfma_f32_16x16x32_bf16 takes its operands (lane l: row l % 16, columns (l / 16) * 8 .. + 7).  Every
// workgroup of a projection reads all of its input rows out of L2, and a load instruction that covers 1 KB of consecutive
// addresses gets 120 GB/s per CU from there (31 TB/s over the chip), one that covers 128 bytes of each of eight rows of
// 8 KB 78, and one that covers 64 bytes of each of sixteen rows 38 (256 workgroups of eight waves that read 0.5 to 18 MB
// in step).  Up to four or eight rows of a one-tile call with packed weights stay row-major (frag false): a k step of a
// single row is then half a line instead of a piece of each of four.  Element index of (row m, column k) in rows of K columns:
__device__ __forceinline__ size_t frag_at(int m, int k, int K) {
  return ((size_t)(m >> 4) * (K >> 5) + (k >> 5)) * 512 + (((k >> 3) & 3) * 16 + (m & 15)) * 8 + (k & 7);
}
__device__ __forceinline__ size_t row_at(bool frag, int m, int k, int K) { return frag ? frag_at(m, k, K) : (size_t)m * K + k; }

// A buffer over `p` for raw buffer loads: 2 GB long, or, where `on` is false, empty (its loads return zeros without a
// memory access, so that a loop's loads need no branch around them past the end).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* p, bool on) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, on ? 0x7fffffff : 0, 0x00020000);
}
// 16 bytes per lane straight from memory to LDS: lane l's go to l * 16 bytes behind `dst`, which is the same in all lanes.
// NT: non-temporal.
template <bool NT = false>
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t buf, char* dst, int lane_offset, int offset) {
#ifdef __HIP_DEVICE_COMPILE__      // (the host pass of the compiler does not know the builtin)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (__attribute__((address_space(3))) void*)dst, 16, lane_offset, offset, 0, NT ? 2 : 0);
#endif
}
// Waits until at most n of the wave's vector memory accesses are outstanding.
#define SP_WAIT_VMEM(n) __builtin_amdgcn_s_waitcnt(0x0f70 | ((n) & 15) | (((n) >> 4) << 14))
// A barrier that waits for no memory access: what has to have arrived is waited for explicitly.  The compiler moves no
// memory access across it.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// max / sum over the four lanes l, l^16, l^32, l^48 (the lanes that share an MFMA column)
__device__ __forceinline__ float quad_rows_max(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_rows_sum(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

template <typename T> struct Elt;
template <> struct Elt<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elt<bf16_t> {
  static __device__ __forceinline__ float ld(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void st(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Sums of squares of up to 16 rows that the kernel producing the rows left as ssq[row][part]: a workgroup of NT threads
// asks for them early (load), adds them up when its products are done (post) and finds the totals in LDS behind the
// barrier that follows.  A wave takes every (NT / 64)-th row; the order of the additions is fixed.
template <int NT>
struct RowSquares {
  static constexpr int NWV = NT / 64, RPW = 16 / NWV;
  f32x4_t v[RPW][2];                               // 512 parts in registers (d_model = 8192); further ones when posting
  __device__ __forceinline__ void load(const float* ssq, int n_part, int M) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int row = wave + i * NWV, p = (j * 64 + lane) * 4;
        v[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
        if (row < M && p < n_part) v[i][j] = *reinterpret_cast<const f32x4_t*>(ssq + (size_t)row * n_part + p);
      }
  }
  __device__ __forceinline__ void post(const float* ssq, int n_part, int M, float* s_tot /* LDS, [16] */) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const int row = wave + i * NWV;
      if (row >= M) continue;
      f32x4_t t = v[i][0] + v[i][1];
      for (int p = (128 + lane) * 4; p < n_part; p += 256)
        t += *reinterpret_cast<const f32x4_t*>(ssq + (size_t)row * n_part + p);
      const float tot = wave_sum((t[0] + t[1]) + (t[2] + t[3]));
      if (lane == 0) s_tot[row] = tot;
    }
  }
};
