// The plan of a forward call: its requests (segments) and the split of its attention work, made on the host.  Plain C++.
#pragma once
#include <stddef.h>

#define SP_BATCH 64       // requests per batched call (== SP_MAX_BATCH_REQ)

enum AttnLoads {
  ATTN_SHARED,             // direct to LDS, staying in the caches
  ATTN_STREAM,             // direct to LDS, non-temporal
  ATTN_STREAM_REGS         // through registers, non-temporal
};

struct AttnPlan {          // host-made split of a forward call's attention work
  int n_seg;
  int qt;                  // 16-row query tiles per workgroup: 1, 2, or 4 (two groups of waves with two tiles each)
  int units_total;         // partial-result units: sum over split segments of chunks * rows * n_q
  int total_items;         // sum over segments of q_blocks * chunks
  int any_split;           // some segment has more than one chunk: the merge kernel must run
  int loads;               // how K/V rows come in (AttnLoads)
  int seg_item0[SP_BATCH]; // first work item of each segment
  int seg_chunks[SP_BATCH];
  int seg_clen[SP_BATCH];  // slots per chunk of the segment (multiple of 32)
  int seg_qblocks[SP_BATCH];
  int seg_unit0[SP_BATCH];
  int seg_row0[SP_BATCH];  // first row of the call that belongs to the segment
  int seg_rows[SP_BATCH];
  int seg_req[SP_BATCH];
  int seg_first[SP_BATCH]; // first node of the segment
  int seg_P[SP_BATCH];     // host mirror of prefix length and live nodes
  int seg_T[SP_BATCH];
  long long seg_base[SP_BATCH];
  void* x_out;             // where the call's result rows go
};

// What the launches of a call depend on beside its number of rows: a captured graph serves the calls for which all of it is equal.
struct AttnShape {
  int qt, items, units, any_split, loads;
  explicit AttnShape(const AttnPlan& p) : qt(p.qt), items(p.total_items), units(p.units_total), any_split(p.any_split), loads(p.loads) {}
  bool operator==(const AttnShape& o) const {
    return qt == o.qt && items == o.items && units == o.units && any_split == o.any_split && loads == o.loads;
  }
};

// Blocks of `per` query rows that the segments make (g query heads of a KV head times the rows).
inline int attn_blocks(const AttnPlan& plan, int g, int per) {
  int n = 0;
  for (int i = 0; i < plan.n_seg; ++i) n += (plan.seg_rows[i] * g + per - 1) / per;
  return n;
}

// Splits every request's cache range into at most `want` chunks; returns the partial-result units that this takes.
inline size_t attn_cut(AttnPlan& plan, int g, int n_q, int want) {
  const int per = 16 * plan.qt;
  size_t units = 0; int items = 0, split = 0;
  for (int i = 0; i < plan.n_seg; ++i) {
    const int span = plan.seg_P[i] + plan.seg_T[i];
    int chunks = want;
    const int max_chunks = (span + 255) / 256;
    if (chunks > max_chunks) chunks = max_chunks;
    if (chunks < 1) chunks = 1;
    const int clen = ((span + chunks - 1) / chunks + 31) / 32 * 32;
    chunks = (span + clen - 1) / clen;
    const int qblocks = (plan.seg_rows[i] * g + per - 1) / per;
    plan.seg_item0[i] = items; plan.seg_chunks[i] = chunks; plan.seg_clen[i] = clen; plan.seg_qblocks[i] = qblocks;
    plan.seg_unit0[i] = (int)units;
    items += chunks * qblocks;
    if (chunks > 1) { units += (size_t)chunks * plan.seg_rows[i] * n_q; split = 1; }
  }
  plan.total_items = items;
  plan.units_total = (int)units;
  plan.any_split = split;
  return units;
}

// The attention work of a plan whose segments are entered, longest cache ranges first: so that the grid fills the chip and the
// partial results fit `room` units.  False: they do not fit.
inline bool attn_split(AttnPlan& plan, int n_q, int n_kv, int n_cu, size_t room) {
  const int g = n_q / n_kv;
  int maxq = 0;
  for (int i = 0; i < plan.n_seg; ++i) if (plan.seg_rows[i] * g > maxq) maxq = plan.seg_rows[i] * g;
  plan.qt = maxq <= 16 ? 1 : 2;
  // Blocks of 64 query rows: half of the tiles' way out of L2, but four runs of slots instead of eight, so that a workgroup takes
  // twice as long, and ranges that a block of 32 would stream by itself are not streamed any more.  They are taken where they
  // are at most two thirds as many as blocks of 32, and not in one round of workgroups of different lengths, whose longest would
  // set the time.  Us a layer of the 8B shape behind 512-4096 slots, blocks of 32 / 64: 31 requests of four nodes and one of nine
  // (33 blocks of 32, 32 of 64; 256 workgroups) 211.4 / 220.3, every second of nine instead of one (48, 32) 212.9 / 225.2, 28
  // requests of 4 and 64 nodes (56, 40) 282.1 / 288.5, 32 of nine (64, 32) 284.4 / 286.9, 32 of 9-16 (64, 32) 315.3 / 322.2; 16 of
  // 24-48 (76, 41; 328 workgroups) 365.1 / 353.8, 64 of 4-12 (99, 64) 444.7 / 438.2, 32 of 8-32 (91, 51) 415.6 / 410.5, two layers of
  // 638 rows (93, 53) 785.0 / 777.1.  One request's ranges are of one length: 70B shape, 256 rows (64, 32; 256) 602.6 / 595.2.
  const int b64 = attn_blocks(plan, g, 64), b32 = attn_blocks(plan, g, 32);
  if (maxq > 32 && 3 * b64 <= 2 * b32 && b64 * n_kv >= (plan.n_seg == 1 ? n_cu : n_cu + n_cu / 4)) plan.qt = 4;
  // One workgroup per CU is the target.  If the query blocks alone give that many, every
  // request keeps its whole cache range in one chunk (no partial results, no merge kernel);
  // otherwise each range is cut into `want` chunks, but never below one 32-slot tile per
  // wave, and fewer if the partial results would not fit the workspace.
  const int wgs = attn_blocks(plan, g, 16 * plan.qt) * n_kv;
  int want = n_cu / wgs;
  // One chunk after all where what the split saves (rounds: 32-slot tiles of the longest range per wave) is not worth the merge,
  // a launch of 4.7 us and the partial rows.  Where no request has a second block, every workgroup streams a range of its own
  // and a tile is a memory latency, 2-2.4 us: two rounds saved are not worth it, three are, or four where half of the CUs
  // stream even uncut.  Blocks that share ranges find them in L2, a tile takes 1-1.2 us, and the more blocks, the more partial
  // rows there are.  Us a layer of the 8B shape, split / whole (workgroups, rounds saved): one row behind 620 and 900 slots (8; 2
  // and 3) 87.6 / 87.6 and 87.3 / 88.8, five requests of one row behind 500, 800 and 1500 (40; 2, 3 and 5) 91.8 / 90.2, 91.2 / 93.2
  // and 94.3 / 98.9, 12 of three behind 1500 (96; 3) 119.7 / 121.7, 16 of one behind 1500 and 2200 (128; 3 and 4) 109.9 / 109.3 and
  // 116.6 / 116.8; 16 rows of one request behind 900 and 1150 (16; 3 and 4) 97.8 / 97.5 and 98.2 / 98.9, 37 behind 700, 1000 and 1450
  // (40; 2, 4 and 5) 120.7 / 117.6, 111.8 / 112.3 and 112.4 / 113.8, 64 behind 1450 and 2000 (64; 4 and 6) 121.4 / 120.1 and 121.6 /
  // 123.3, 128 behind 2200, 2700 and 3400 (128; 5, 6 and 7) 152.9 / 152.0, 154.3 / 153.9 and 155.1 / 156.0, four requests of 24 behind
  // 1700 and 3000 (96; 3 and 6) 135.3 / 133.0 and 138.7 / 139.6.
  if (want > 1) {
    int longest = 0;
    bool shared = false;
    for (int i = 0; i < plan.n_seg; ++i) {
      longest = plan.seg_P[i] + plan.seg_T[i] > longest ? plan.seg_P[i] + plan.seg_T[i] : longest;
      shared = shared || plan.seg_rows[i] * g > 16 * plan.qt;
    }
    const int rounds = (longest + 255) / 256, saved = rounds - (rounds + want - 1) / want;
    if (shared ? 2 * saved <= 5 + 16 * wgs / n_cu : saved <= (2 * wgs < n_cu ? 2 : 3)) want = 1;
  }
  size_t units = attn_cut(plan, g, n_q, want);
  while (units > room && want > 1) { want = (want + 1) / 2; units = attn_cut(plan, g, n_q, want); }
  if (units > room) return false;
  // K/V rows are read once where every request is one block.  Through registers where one workgroup per request streams ranges of
  // different lengths: the longest ones set the time, alone on their CUs, and a tile that waits in registers keeps their loads in
  // flight all the time (32 requests of 512-4096 slots 58.8 us, direct to LDS 65.4).  One request, or ranges cut into chunks:
  // every CU streams, and direct-to-LDS loads are level or faster (two to sixteen requests of a few rows, whole steps 0.5-2 %).
  plan.loads = ATTN_STREAM;
  for (int i = 0; i < plan.n_seg; ++i) if (plan.seg_qblocks[i] > 1) plan.loads = ATTN_SHARED;
  if (plan.loads == ATTN_STREAM && plan.n_seg > 1 && !plan.any_split) plan.loads = ATTN_STREAM_REGS;
  return true;
}
