// Host functions and plan fields that decide what the kernels read, how they are split and which of
// them runs, for tests/test_plan_rules_cpu.py (compiled there, takes handles of the library's set-up).
#include "internal.h"

extern "C" {

int64_t probe_slice_bytes(int64_t rows, int64_t ld, int64_t f4, int64_t c4) {
  return pgcn::slice_bytes(rows, ld, f4, c4);
}

void probe_tn_split(int K, int tiles, int splits, int slab, int *out) {
  const pgcn::TnSplit r = pgcn::tn_split(K, tiles, splits, slab);
  out[0] = r.splits;
  out[1] = r.chunk;
}

int probe_pack_by_row(int64_t count, int64_t rows, int64_t f4, int64_t ld, int64_t dst) {
  return pgcn::pack_by_row(count, rows, f4, ld, (const void *)dst);
}

// out: chunks, partial slots, whole_bytes, full_bytes (-1: never), then the column cuts of plan
// `which` (0 plain, 1 narrow, 2 sliced; chunks 0: none); returns the number of values.
int probe_plan(const pgcn_partition *p, int transposed, int which, int64_t *out) {
  const pgcn::Plan *f[3] = {&p->plan, &p->plan_n, &p->plan_s}, *t[3] = {&p->plan_t, &p->plan_tn, &p->plan_ts};
  const pgcn::Plan &q = *(transposed ? t : f)[which];
  int n = 0;
  out[n++] = q.chunks;
  out[n++] = q.slots;
  out[n++] = q.use.whole_bytes == pgcn::kNever ? -1 : q.use.whole_bytes;
  out[n++] = q.use.full_bytes == pgcn::kNever ? -1 : q.use.full_bytes;
  if (q.chunks > 0)
    for (int64_t c : q.chunk_cols) out[n++] = c;
  return n;
}

// 0, 1 or 2 (as above): the plan that an aggregation of f floats from sources at lo and hi runs.
int probe_taken(const pgcn_partition *p, int transposed, int64_t f, int64_t lo, int64_t hi, int64_t ld) {
  const pgcn::Plan &q = pgcn::agg_plan(p, transposed != 0, f, (const float *)lo, (const float *)hi, ld);
  if (q.sliced) return 2;
  return &q == &p->plan || &q == &p->plan_t ? 0 : 1;
}

}  // extern "C"
