// C entries to the library's scoring-range arithmetic, for the tests without a GPU.
#include "ckv_device.hpp"

extern "C" {
int t_stage_rows() { return ckv::kStageRows; }
int t_max_partials() { return ckv::kMaxPartials; }
int t_claim_rows() { return ckv::kClaimGroups * ckv::kStageRows; }
uint32_t t_groups_of(int n) { return ckv::groups_of(n); }
int t_static_rows(int n) { return ckv::static_rows(n); }
uint32_t t_range_groups(uint32_t total, int nwg, int min_range) {
  return ckv::range_groups(total, nwg, min_range);
}
void t_range_of(int wg, uint32_t R, uint32_t total, uint32_t* out) {
  const ckv::GroupRange r = ckv::range_of(wg, R, total);
  out[0] = r.g0;
  out[1] = r.g1;
}
int t_min_range_groups(int64_t gu, int slots) { return ckv::min_range_groups(gu, slots); }
int t_added_min_range(int64_t gu) { return ckv::added_min_range(gu); }
void t_unit_ranges(uint32_t before, uint32_t mine, uint32_t R, uint32_t* out) {
  const ckv::UnitRanges r = ckv::unit_ranges(before, mine, R);
  out[0] = r.first;
  out[1] = r.count;
}
int t_slots_fit(int64_t gu, int64_t units, int nwg, int slots) {
  return ckv::slots_fit(gu, units, nwg, slots);
}
}
