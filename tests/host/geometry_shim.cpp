// C entry points over the library's host-side geometry (csrc/geometry.h), for the tests.
#include "geometry.h"

extern "C" {

// out: grid, count_groups, send_groups, senders, batch, combine_run.
void plan_decomposed(int R, int E, int k, int Tr, int H, int count_groups, int sync, int capacity, int cus, int* out) {
  const epl::DecomposedPlan p = epl::split_decomposed(epl::make_geom(R, E, k, Tr), H, count_groups, sync, capacity, cus);
  const int v[] = {p.grid, p.count_groups, p.send_groups, p.senders, p.batch, p.combine_run};
  for (int i = 0; i < 6; ++i) out[i] = v[i];
}

unsigned unit_grid(int64_t units, int per_group, int threads) { return epl::unit_grid(units, per_group, threads); }

}  // extern "C"
