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

}  // extern "C"
