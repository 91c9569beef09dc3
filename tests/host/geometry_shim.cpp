// C entry points over the library's host-side geometry (csrc/geometry.h), for the tests.
#include "geometry.h"

extern "C" {

int decomposed_form(int R, int E, int k, int Tr, int H, int sync) {
  return epl::decomposed_form(epl::make_geom(R, E, k, Tr), H, sync);
}

// out: grid, count_groups, send_groups, senders, batch, combine_run.
void plan_decomposed(int R, int E, int k, int Tr, int H, int count_groups, int sync, int form, int capacity, int cus,
                     int* out) {
  const epl::DecomposedPlan p =
      epl::split_decomposed(epl::make_geom(R, E, k, Tr), H, count_groups, sync, form, capacity, cus);
  const int v[] = {p.grid, p.count_groups, p.send_groups, p.senders, p.batch, p.combine_run};
  for (int i = 0; i < 6; ++i) out[i] = v[i];
}

// out: of the layout's chunking CT, NC, nblk; of the chunks route_place launches the same; place_sum of
// these; whether place_layout takes the layout.
void layout_chunks(int R, int E, int k, int Tr, int* out) {
  const epl::Geom g = epl::make_geom(R, E, k, Tr);
  const epl::Geom p = epl::place_geom(g);
  const int v[] = {g.CT, g.NC, g.nblk, p.CT, p.NC, p.nblk, (int)std::min<int64_t>(epl::place_sum(p), INT_MAX),
                   epl::place_layout(g)};
  for (int i = 0; i < 8; ++i) out[i] = v[i];
}

// The most pairs in the group rows that one thread of route_place adds up, counted chunk by chunk.
int place_sum_counted(int R, int E, int k, int Tr) {
  const epl::Geom p = epl::place_geom(epl::make_geom(R, E, k, Tr));
  int64_t sum[epl::kPlaceRows] = {};
  for (int b = 0; b < p.nblk; ++b) {
    const int c = b % p.NC;
    sum[b / epl::kGroupChunks % epl::kPlaceRows] += (int64_t)std::max(0, std::min(p.CT, Tr - c * p.CT)) * k;
  }
  return (int)std::min<int64_t>(*std::max_element(sum, sum + epl::kPlaceRows), INT_MAX);
}

int small_dispatch(int R, int E, int k, int Tr, int H, int fp8) {
  return epl::small_dispatch(epl::make_geom(R, E, k, Tr), H, fp8 != 0);
}

int long_slices(int64_t pairs, int H, int64_t slices) {
  return epl::long_slices(pairs, H, (H / 8 + 255) / 256, slices);
}

unsigned unit_grid(int64_t units, int per_group, int threads) { return epl::unit_grid(units, per_group, threads); }

}  // extern "C"
