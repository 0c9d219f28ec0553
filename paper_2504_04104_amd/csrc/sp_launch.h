// Host-callable launchers of the HIP kernels.  Each enqueues on `st` and returns
// the launch status; none synchronises.
#pragma once
#include "sp_device.h"

struct KvGeom {
  char* kv;              // slab
  size_t plane_bytes;    // bytes between consecutive kv heads: kv_slots * row_bytes
  int row_bytes;         // d_head * element size
  int n_layers;
  int n_kv_heads;
  // Paged storage (SpecPipe-DB keeps its cache in pages, Sec. 4 "Implementation"): request r's
  // logical slot s lives in physical slot page_table[r * pt_stride + (s >> pg_shift)] << pg_shift
  // | (s & mask).  Null: a request owns the contiguous range that starts at its base slot.
  int* page_table;
  int pt_stride;
  int pg_shift;
};

// Physical slot of a request's logical slot (base is the request's first slot when contiguous, 0 when paged).
__device__ __forceinline__ size_t sp_phys_slot(const KvGeom& g, int req, long long base, int lslot) {
  if (!g.page_table) return (size_t)(base + lslot);
  const int page = g.page_table[(size_t)req * g.pt_stride + (lslot >> g.pg_shift)];
  return ((size_t)page << g.pg_shift) | (size_t)(lslot & ((1 << g.pg_shift) - 1));
}

// ---- tree tables -------------------------------------------------------------
hipError_t sp_launch_tables_clear(ReqMeta* meta, ReqTables* tables, int n_req, hipStream_t st);
hipError_t sp_launch_request_init(ReqMeta* meta, ReqTables* tables, int req, long long base, int cap, int P,
                                  hipStream_t st);
// first_slot: cache slot of the first new node (host mirror: base + prefix_len + n_live)
hipError_t sp_launch_tree_insert(ReqMeta* meta, ReqTables* tables, const InsertArgs& a, KvGeom g, hipStream_t st);
// dev_nodes (nullable, device): item i accepts node dev_nodes[i * dev_stride] if it is a live node and clears
// the tree otherwise; the modes and nodes of `b` are then ignored (entries with mode < 0 are still skipped)
hipError_t sp_launch_tree_prune(ReqMeta* meta, ReqTables* tables, const PruneBatch& b, const int* dev_nodes,
                                int dev_stride, hipStream_t st);
hipError_t sp_launch_pages_set(int* page_table, int pt_stride, int req, int first, int n, const int* pages /*host*/,
                               hipStream_t st);
// out[i] (device) = verified root child of request reqs[i], or -1
hipError_t sp_launch_tree_match(const ReqMeta* meta, const ReqTables* tables, int n, const int* reqs, int* out,
                                hipStream_t st);
hipError_t sp_launch_tree_expand(const ReqTables* tables, const ExpandArgs& a, const int* cand_tok,
                                 const float* cand_prob, int* out_parent, int* out_token, float* out_prob,
                                 int* out_count, hipStream_t st);
hipError_t sp_launch_set_root_pred(ReqMeta* meta, int req, int token, hipStream_t st);

// ---- lossy verification (sp_verify.hip) -------------------------------------------
// xn = rmsnorm(x) * gain for M rows (no residual stream, no row descriptors)
hipError_t sp_launch_row_norm(int dtype, const void* x, const void* gain, void* xn, bool frag, int M, int d, float eps,
                              hipStream_t st);
// floats of scratch sp_launch_verify_lossy needs at least for n rows of V logits (it uses more if there is more)
size_t sp_lossy_scratch_floats(int n, int V);
// Logits of n rows whose products were formed in tiles of tile_cols columns (0: none) lie as [n][V] or, tiles of this many
// columns, as [V / columns][n][columns].
static inline int logits_lie(int tile_cols) { return tile_cols == 128 ? 128 : 0; }
// mode 1 relaxed, 2 top-p; out[2i] = verified node of reqs[i] or -1, out[2i+1] = top-1 token
hipError_t sp_launch_verify_lossy(ReqMeta* meta, const ReqTables* tables, const float* logits, int tile_cols, int n, const int* reqs,
                                  int V, int mode, float top_p, float* scratch, size_t scratch_floats, int* out,
                                  hipStream_t st);
// stochastic verification: out[2i] = verified node of reqs[i] or -1, out[2i+1] = the token drawn at u[i]
hipError_t sp_launch_verify_sample(ReqMeta* meta, const ReqTables* tables, const float* logits, int n, const int* reqs,
                                   int V, float temperature, float top_p, int top_k, const float* u /*host*/,
                                   const float* stats /*nullable: sp_launch_gemm_logits_bf16's*/, int tile_cols, int* out,
                                   hipStream_t st);
hipError_t sp_launch_kv_compact(const ReqMeta* meta, const ReqTables* tables, const PruneBatch& b, KvGeom g,
                                void* rows /*nullable: hidden rows of the one request, same launch*/,
                                size_t row_stride_bytes, int row_bytes, const RowList* l, hipStream_t st);

// ---- elementwise / row kernels --------------------------------------------------
// Rows enter the stage: row descriptors and rotary tables (cs: [rows][d_head], cos then sin),
// h = x, xn = rmsnorm(h) * gain (frag, bf16 only: in fragment order, as every bf16 matrix-core product reads its rows).
// The segment fields of `plan` say which request and node each row belongs to; if plan_dev is given the
// whole plan is also stored there for the attention kernels of the call.
hipError_t sp_launch_enter_norm(int dtype, const void* x, const AttnPlan& plan, AttnPlan* plan_dev /*nullable*/,
                                const ReqMeta* meta, const ReqTables* tables, RowInfo* rows, float* cs, int d_head,
                                float theta, float* h, const void* gain, void* xn, bool frag, int M, int d, float eps,
                                hipStream_t st);

// h += sum_s part[s]; xn = rmsnorm(h) * gain
hipError_t sp_launch_add_norm(int dtype, float* h, const float* part, int S, size_t part_stride,
                              const void* gain, void* xn, bool frag, int M, int d, float eps, hipStream_t st);
// q,k rotated, v copied; q -> qbuf [M][n_q*d_head]; k,v -> slab rows
hipError_t sp_launch_rope_kv(int dtype, const float* part, int S, size_t part_stride, const RowInfo* rows,
                             const float* cs, void* qbuf, KvGeom g, int layer, int M, int n_q, int n_kv,
                             int d_head, hipStream_t st);
// top-1 token per row from per-tile (value, index) pairs or from plain logits; also written to tables[..].pred
hipError_t sp_launch_argmax_rows(bool pairs, const float* part, int n_items, const FwdBatch& b, ReqTables* tables,
                                 int* pred_out /*nullable*/, float* max_out /*nullable*/, hipStream_t st);
hipError_t sp_launch_silu_mul(int dtype, const float* gu, void* act, int M, int F, hipStream_t st);
// plan_dev (nullable): the call's plan on the device; its x_out then takes the place of `out`
hipError_t sp_launch_finish(int dtype, const float* h, const float* part, int S, size_t part_stride, void* out,
                            const AttnPlan* plan_dev, int M, int d, hipStream_t st);

// ---- GEMM: out[s][m][n] (f32) = sum over the s-th K slice of X[m][k] * W[n][k] -----
hipError_t sp_launch_gemm_simple(int dtype, const void* X, const void* W, float* out, int M, int N, int K,
                                 hipStream_t st);
// float32 on the matrix cores (K % 4 == 0, rows 16-byte aligned)
hipError_t sp_launch_gemm_f32(const float* X, const float* W, float* out, int M, int N, int K, hipStream_t st);
// the float32 layer's products with what stands before and after them (h: the residual stream [M][d], float32):
// qkv of rmsnorm(h), rotated, to qbuf and the cache; silu(gate) * up of rmsnorm(h); h += X W^T, or with plan_out the plan's
// x_out = h + X W^T
bool sp_qkv_f32_joined(int M, int N, int n_cu);       // else: a norm, sp_launch_gemm_f32 and a rotation of their own
hipError_t sp_launch_qkv_f32(const float* h, const float* gain, float eps, const float* W, const RowInfo* rows, const float* cs,
                             float* qbuf, KvGeom g, int layer, int M, int d, int n_q, int n_kv, int d_head, hipStream_t st);
hipError_t sp_launch_gateup_f32(const float* h, const float* gain, float eps, const float* W, float* act, int M, int F, int K,
                                hipStream_t st);
hipError_t sp_launch_residual_f32(const float* X, const float* W, float* h, const AttnPlan* plan_out /*nullable*/, int M, int N,
                                  int K, hipStream_t st);
hipError_t sp_launch_attn_f32(const float* q, const RowInfo* rows, const ReqTables* tables, KvGeom g, int layer, float* out,
                              int M, int n_q, int n_kv, int d_head, hipStream_t st);
// bf16 MFMA kernels: the rows X and the gate/up products are in fragment order (frag_at).  Up to 64 rows.  Returns the split
// count used in *S_out (partials [S][M][N]).  packed: the weights are in MFMA fragment order (sp_launch_pack_weights).  frag
// false: X is row-major, as it has to be beside row-major weights, and may be up to eight rows beside packed ones.
hipError_t sp_launch_gemm_bf16(const bf16_t* X, const bf16_t* W, bool packed, float* out, int M, int N, int K,
                               int max_split, size_t part_capacity_floats, int* S_out, hipStream_t st,
                               bool resident, bool frag);
// Logits (in tiles; stats nullable) and output head: X in fragment order beside packed weights, row-major beside row-major ones.
hipError_t sp_launch_gemm_logits_bf16(const bf16_t* X, const bf16_t* W, bool packed, float* logits, float* stats, float inv_T,
                                      int M, int V, int K, int* tile_cols, hipStream_t st);
// act[m][f] = silu(X Wg^T) * (X Wu^T), W = [gate rows ; up rows]
hipError_t sp_launch_gemm_argmax_bf16(const bf16_t* X, const bf16_t* W, bool packed, float* pairs, int M, int V, int K,
                                      size_t pair_capacity_floats, int* tiles_out, hipStream_t st);
// ssq (nullable, M <= 16 only): [M][K / 16] sums of squares of the rows, X is then not normalised yet.  frag false (M <= 16
// only): X and the products are row-major.
hipError_t sp_launch_gemm_gateup_bf16(const bf16_t* X, bool frag, const bf16_t* W, bool packed, bf16_t* act, int M, int F,
                                      int K, int n_cu, const float* ssq, float eps, hipStream_t st);
// One row tile (M <= 16), fast path: complete projections with what follows them as their epilogue (sp_gemm_few.hip);
// `takes` says for which sizes these are to be called (d = d_model, dq = n_q * d_head).  frag: how X and the rows left for
// the next product lie.
bool sp_few_takes(int M, int d, int dq, int F, bool packed, int n_cu);
// ssq (nullable): [M][d / 16] sums of squares of the rows, X is then not normalised yet.
hipError_t sp_launch_few_qkv(const bf16_t* X, bool frag, const bf16_t* W, bool packed, const float* ssq, float eps, const RowInfo* rows,
                             const float* cs, bf16_t* qbuf, KvGeom g, int layer, int M, int K, int n_q, int n_kv,
                             int n_cu, hipStream_t st);
// h += X W^T; xn = bf16(h * gain); ssq_out[M][N / 16]
hipError_t sp_launch_few_residual(const bf16_t* X, bool frag, const bf16_t* W, bool packed, bool resident, float* h, const bf16_t* gain,
                                  bf16_t* xn, float* ssq_out, int M, int N, int K, int n_cu,
                                  hipStream_t st);
// rows of the plan's x_out = bf16(h + X W^T)
hipError_t sp_launch_few_out(const bf16_t* X, bool frag, const bf16_t* W, bool packed, const float* h, const AttnPlan* plan_dev, int M,
                             int N, int K, int n_cu, hipStream_t st);
// Up to 160 rows, gate/up 192 (sp_gemm_mid.hip): one workgroup per CU, two strips of weight rows per wave, X in fragment
// order; `takes` says for which sizes these are to be called (gate/up: where every CU gets the same 49-64 or 97-112 columns)
bool sp_gemm_mid_takes(int M, int N, int K, bool packed, int n_cu);
bool sp_gemm_mid_takes_gateup(int M, int F, int K, bool packed, int n_cu);
hipError_t sp_launch_gemm_mid(const bf16_t* X, const bf16_t* W, bool packed, float* out, int M, int N, int K, int n_cu,
                              int max_split, size_t part_capacity_floats, int* S_out, hipStream_t st, bool resident);
hipError_t sp_launch_gemm_mid_gateup(const bf16_t* X, const bf16_t* W, bool packed, bf16_t* act, int M, int F, int K, int n_cu,
                                     const float* ssq, float eps, hipStream_t st);
// Many rows (more than the kernels above take): workgroups of 128 or 256 rows x 256 columns, weights kept in registers per wave.
// Needs N % 256 == 0 (gate/up: F % 128 == 0) and K % 64 == 0.
hipError_t sp_launch_gemm_wide(const bf16_t* X, bool frag, const bf16_t* W, bool packed, float* out, int M, int N, int K,
                               int n_cu, size_t part_capacity_floats, int* S_out, hipStream_t st);
hipError_t sp_launch_gemm_wide_gateup(const bf16_t* X, bool frag, const bf16_t* W, bool packed, bf16_t* act, int M, int F, int K,
                                      int n_cu, hipStream_t st);
// [N][K] row-major bf16 -> MFMA fragment order (N % 16 == 0, K % 32 == 0, out != in)
hipError_t sp_launch_pack_weights(const void* in, void* out, int N, int K, hipStream_t st);

// ---- tree attention -------------------------------------------------------------
hipError_t sp_launch_attn_simple(int dtype, const void* q, const RowInfo* rows, const ReqTables* tables, KvGeom g,
                                 int layer, void* out, int M, int n_q, int n_kv, int d_head, hipStream_t st);

// plan: host copy (grid sizes); plan_dev: the device copy the kernels read
hipError_t sp_launch_attn_bf16(const bf16_t* q, const ReqTables* tables, KvGeom g, int layer, const AttnPlan& plan,
                               const AttnPlan* plan_dev, float* part /*workspace*/, bf16_t* out, bool frag, int M,
                               int n_q, int n_kv, int d_head, hipStream_t st);
