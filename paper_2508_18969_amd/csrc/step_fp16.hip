// The fused chemistry-update kernel instantiated for FP16 operands.
#include "step_small.h"

namespace chemdnn {

// Compiled network shapes: the 17-species net (400, 200, 100) and the
// 29-species net (1600, 800, 400).
bool find_layout_fp16(int h1, int h2, int h3, NetLayout *out) {
  if (h1 == 400 && h2 == 200 && h3 == 100) {
    fill_small_layout<Cfg<OpF16, 4, 4, 400, 200, 100>, false, 4>(out);
    return true;
  }
  if (h1 == 1600 && h2 == 800 && h3 == 400) {
    fill_layout<Cfg<OpF16, 4, 8, 1600, 800, 400>, false>(out);
    return true;
  }
  return false;
}

// Property mode: the density network of the supercritical flame,
// 3-1024-512-256-1 (its 1.35 MB of BF16 weights fit the L2 of an XCD).  Tiles of
// 64 cells, or of 48 where these fill the rounds better: 300 / 12,288 / 16,384 /
// 20,011 cells take 24.0 / 27.7 / 29.0 / 49.0 us in the first, 22.2 / 26.8 / 44.9 /
// 45.2 in the second (a round 21.6 and 18.6).
bool find_prop_layout_fp16(int h1, int h2, int h3, NetLayout *out) {
  if (h1 == 1024 && h2 == 512 && h3 == 256) {
    using Large = Cfg<OpF16, 4, 8, 1024, 512, 256>;
    using Small = Cfg<OpF16, 3, 8, 1024, 512, 256>;
    static_assert(Large::R2 == Small::R2 && Large::R3 == Small::R3 && Large::NQ3 == Small::NQ3 &&
                  Large::NQ4 == Small::NQ4, "one packed layout");
    fill_prop_layout<Large>(out);
    out->pick[0] = [](const StepArgs &a, int n_cu, hipStream_t s) {
      return launch_by_size<Large, Small, true>(a, n_cu, {7400, 21600}, {8200, 18600}, s);
    };
    out->pick_prepare[0] = prepare_prop<Small>;
    return true;
  }
  return false;
}

}  // namespace chemdnn
