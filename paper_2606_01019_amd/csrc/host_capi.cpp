// Host-only C entry points over HostState, built with the system C++ compiler
// (no HIP) so the page allocator and verify/commit state machine can be
// tested on a machine without a GPU.
#include <stdint.h>

#include <cstring>

#include "host_state.h"
#include "attn_order.h"
#include "mid_plan.h"
#include "tiled_plan.h"

using hvd::HostState;

extern "C" {

void* hvdh_create(int32_t max_seqs, int32_t n_pages, int32_t max_pos, int32_t max_draft, int32_t vocab) {
  return new HostState(max_seqs, n_pages, 16, max_pos, max_draft, vocab);
}
void hvdh_destroy(void* h) { delete (HostState*)h; }
int hvdh_prefill(void* h, int32_t id, const int32_t* toks, int32_t n) { return ((HostState*)h)->begin_prefill(id, toks, n); }
int hvdh_begin_verify(void* h, int32_t batch, const int32_t* ids, const int32_t* ctx, const int32_t* draft,
                      const int32_t* lens) {
  return ((HostState*)h)->begin_verify(batch, ids, ctx, draft, lens);
}
void hvdh_finish_verify(void* h, int32_t batch, const int32_t* ids, const int32_t* draft, const int32_t* lens,
                        const int32_t* acc, const int32_t* next) {
  ((HostState*)h)->finish_verify(batch, ids, draft, lens, acc, next);
}
void hvdh_abort_verify(void* h, int32_t batch, const int32_t* ids) { ((HostState*)h)->abort_verify(batch, ids); }
int hvdh_commit(void* h, int32_t batch, const int32_t* ids, const int32_t* keep) {
  return ((HostState*)h)->commit(batch, ids, keep);
}
int hvdh_begin_async(void* h, int32_t batch, const int32_t* ids, const int32_t* ctx, const int32_t* lens,
                     int32_t max_steps) {
  return ((HostState*)h)->begin_async(batch, ids, ctx, lens, max_steps);
}
void hvdh_end_async(void* h, int32_t batch, const int32_t* ids, const int32_t* ctx, const int32_t* pend) {
  ((HostState*)h)->end_async(batch, ids, ctx, pend);
}
int hvdh_truncate(void* h, int32_t id, int32_t ctx, int32_t pend) { return ((HostState*)h)->truncate(id, ctx, pend); }
int hvdh_free_seq(void* h, int32_t id) { return ((HostState*)h)->free_seq(id); }
int32_t hvdh_free_pages(void* h) { return ((HostState*)h)->free_pages(); }
// ctx, pending, verify_pending, number of pages; -1 if not live
int hvdh_seq(void* h, int32_t id, int32_t* out4) {
  const HostState* s = (const HostState*)h;
  if (id < 0 || id >= s->max_seqs() || !s->seq(id).live) return -1;
  const auto& q = s->seq(id);
  out4[0] = q.ctx;
  out4[1] = q.pending;
  out4[2] = q.verify_pending ? 1 : 0;
  out4[3] = (int32_t)q.pages.size();
  return 0;
}
// copies up to cap page ids of seq id; returns the count
int32_t hvdh_pages(void* h, int32_t id, int32_t* out, int32_t cap) {
  const auto& q = ((HostState*)h)->seq(id);
  int32_t n = (int32_t)q.pages.size();
  for (int32_t i = 0; i < n && i < cap; ++i) out[i] = q.pages[i];
  return n;
}
const char* hvdh_error(void* h) { return ((HostState*)h)->error().c_str(); }

// Whether gemm_mid takes a GEMM, and its plan: strips, splits, row blocks, row tiles per block
int hvdh_mid_plan(int32_t mtiles, int32_t N, int32_t K, int32_t wide, int64_t part_bytes, int32_t f_strips,
                  int32_t f_splits, int32_t* out4) {
  const int force[2] = {f_strips, f_splits};
  const hvd::MidPlan p = hvd::mid_plan(mtiles, N / 16, K / 32, 192, wide != 0, (size_t)part_bytes, force);
  out4[0] = p.strips;
  out4[1] = p.splits;
  out4[2] = p.mblocks;
  out4[3] = p.mt_block;
  return hvd::mid_takes(mtiles, N, K);
}
// Work plan of a large-batch GEMM: tile, workgroups, shared tiles, sharing workgroups
void hvdh_tiled_plan(int32_t mtiles, int32_t N, int32_t KT, int32_t single, int32_t cus, int64_t part_bytes, int32_t* out4) {
  const hvd::TiledPlan p = hvd::tiled_plan(mtiles, N, KT, single != 0, cus, (size_t)part_bytes);
  out4[0] = p.tile;
  out4[1] = p.n_wg;
  out4[2] = p.n_shared;
  out4[3] = p.n_sk;
}
int hvdh_tiled_plan_ok(int32_t tile, int32_t n_wg, int32_t n_shared, int32_t n_sk, int32_t T, int32_t KT) {
  return hvd::tiled_plan_ok(hvd::TiledPlan{tile, n_wg, n_shared, n_sk}, T, KT);
}
// Run of worker w ([out4[0], out4[1])), the worker of the w-th workgroup, and the holder of step lo(w)
void hvdh_tiled_run(int32_t n_shared, int32_t KT, int32_t n_sk, int32_t w, int32_t* out4) {
  const hvd::SharedRuns r(n_shared, KT, n_sk);
  out4[0] = r.lo(w);
  out4[1] = r.lo(w + 1);
  out4[2] = r.worker(w);
  out4[3] = r.holder(r.lo(w));
}
// Partial slot of worker w's part of shared tile t
int32_t hvdh_tiled_slot(int32_t n_shared, int32_t KT, int32_t n_sk, int32_t w, int32_t t) {
  return hvd::SharedRuns(n_shared, KT, n_sk).slot0(w) + t;
}
// Launch order of attention items [n][4] (stream, unit, chunk, keys), longest first or
// interleaved; returns the count, no-op pieces (unit -1) included
static int32_t attn_pieces(bool longest_first, int32_t n, const int32_t* in, int32_t* out, int32_t cap) {
  std::vector<hvd::AttnPiece> p(n);
  for (int32_t i = 0; i < n; ++i) p[i] = {in[4 * i], in[4 * i + 1], in[4 * i + 2], in[4 * i + 3]};
  p = longest_first ? hvd::attn_order(p) : hvd::attn_interleave(p);
  for (size_t i = 0; i < p.size() && (int32_t)i < cap; ++i) {
    out[4 * i] = p[i].stream;
    out[4 * i + 1] = p[i].unit;
    out[4 * i + 2] = p[i].chunk;
    out[4 * i + 3] = p[i].keys;
  }
  return (int32_t)p.size();
}
// Whether the launch gains from the longest-first order
int hvdh_attn_order_pays(int32_t n, const int32_t* in, int32_t cus) {
  std::vector<hvd::AttnPiece> p(n);
  for (int32_t i = 0; i < n; ++i) p[i] = {in[4 * i], in[4 * i + 1], in[4 * i + 2], in[4 * i + 3]};
  return hvd::attn_order_pays(p, cus);
}
int32_t hvdh_attn_order(int32_t n, const int32_t* in, int32_t* out, int32_t cap) {
  return attn_pieces(true, n, in, out, cap);
}
int32_t hvdh_attn_interleave(int32_t n, const int32_t* in, int32_t* out, int32_t cap) {
  return attn_pieces(false, n, in, out, cap);
}
}
