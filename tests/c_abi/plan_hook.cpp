// What a test may ask about the plan of a problem: where the block of approximate cosines, the unit rows, the text
// profiles and their maxima lie in the workspace, how the block is cut, and the error its readers allow for; how the reduction
// of the maps is cut; the order of causal tiles; the form of the feature passes.  (Host code only.)
#include "../../paper_2411_17686_amd/csrc/common.hpp"
#include "../../paper_2411_17686_amd/csrc/causal_tiles.hpp"

extern "C" {

struct gram_plan {
  int64_t ct, xhat, ttext, cmax;   // byte offsets in the workspace
  int32_t use_gram, splits;  // K ranges: [splits][B][n_disc][n_keep]
  int32_t st_per_split, form, Df;
  float delta;
};

// Status of ficoco.h.
int plan_hook_gram(const ficoco_problem* p, gram_plan* out) {
  ficoco::Plan pl{};
  const char* why = nullptr;
  const int rc = ficoco::make_plan(*p, pl, &why);
  if (rc != FICOCO_OK) return rc;
  *out = gram_plan{(int64_t)pl.ct, (int64_t)pl.xhat, (int64_t)pl.ttext, (int64_t)pl.cmax, pl.use_gram, pl.gram_splits, pl.gram_st_per_split,
                   pl.use_gram ? (int32_t)ficoco::gram_form(*p, pl) : 0, pl.Df, ficoco::gram_delta(pl)};
  return rc;
}

struct reduce_plan {
  int64_t total, beyond;     // bytes of the workspace; those that the limit of the static scratch does not count
  int32_t row_lanes, strip_groups, rows, chunks, combined;
};

// scratch: as in make_plan
int plan_hook_reduce(const ficoco_problem* p, uint64_t scratch, reduce_plan* out) {
  ficoco::Plan pl{};
  const char* why = nullptr;
  const int rc = ficoco::make_plan(*p, pl, &why, scratch);
  if (rc != FICOCO_OK) return rc;
  *out = reduce_plan{(int64_t)pl.total, (int64_t)pl.beyond, pl.row_lanes, pl.strip_groups, pl.rows_per_wg, pl.n_chunks, ficoco::partials_combined(*p, pl)};
  return rc;
}

int plan_hook_unit_rows_summed(const ficoco_problem* p) { return ficoco::unit_rows_summed(*p, p->F ? p->Df : p->D); }
int plan_hook_causal_long_first(int first, int last) { return ficoco::causal_long_first(first, last); }
int plan_hook_causal_live_first(int units, int k_tiles) { return ficoco::causal_live_first(units, k_tiles); }

// The order of all groups x k_tiles tiles: group and key tile of each.
void plan_hook_causal_tiles(int groups, int k_tiles, int per, int full, int32_t* out) {
  for (int unit = 0; unit < groups * k_tiles; ++unit) ficoco::causal_tile(unit, groups, k_tiles, per, full, out[2 * unit], out[2 * unit + 1]);
}

}  // extern "C"
