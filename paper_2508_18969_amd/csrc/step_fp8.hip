// The fused chemistry-update kernel instantiated for FP8 E4M3 operands.
#include "step_small.h"

namespace chemdnn {

// The 29-species net in tiles of 64 cells (25 accumulator tiles per wave, 71
// registers spilled; 39 us a round) and of 48 (none spilled; 32 us): a round of
// either costs about the same per cell, so the smaller ones are for batches
// whose rounds they fill better.  16 / 12,288 / 16,384 / 20,000 / 300,007 cells,
// us: 64-cell tiles 46 / 52 / 55 / 93 / 760, 48-cell tiles 37 / 44 / 75 / 75 / 817.
// The tabulated GELU always takes 48 (131,072 cells 587 us against 792).
using Large29 = Cfg<OpF8, 4, 8, 1600, 800, 400>;
using Small29 = Cfg<OpF8, 3, 8, 1600, 800, 400>;
static_assert(Large29::R2 <= Small29::R2 && Large29::R3 <= Small29::R3 && Large29::NQ2 == Small29::NQ2 &&
              Large29::NQ3 == Small29::NQ3 && Large29::NQ4 == Small29::NQ4, "one packed layout");
constexpr TileTime kTime29L = {16000, 39000}, kTime29S = {12000, 32000};

// Compiled network shapes: the 17-species net (400, 200, 100) and the
// 29-species net (1600, 800, 400).
bool find_layout_fp8(int h1, int h2, int h3, NetLayout *out) {
  if (h1 == 400 && h2 == 200 && h3 == 100) {
    fill_small_layout<Cfg<OpF8, 3, 4, 400, 200, 100>, false, 4>(out);
    return true;
  }
  if (h1 == 1600 && h2 == 800 && h3 == 400) {
    fill_layout<Small29, false>(out);
    out->pick[0] = [](const StepArgs &a, int n_cu, hipStream_t s) {
      return launch_by_size<Large29, Small29, false>(a, n_cu, kTime29L, kTime29S, s);
    };
    out->pick_prepare[0] = [] { return set_lds_limit<Large29, false, 0>(); };
    out->pick_dbg = [](const StepArgs &a, int n_cu, hipStream_t s) {
      return launch_by_size<Large29, Small29, false, true>(a, n_cu, kTime29L, kTime29S, s);
    };
    out->pick_dbg_prepare = [] { return set_lds_limit<Large29, false, 0, false, true>(); };
    out->pick_species = 30;
    return true;
  }
  return false;
}

}  // namespace chemdnn
