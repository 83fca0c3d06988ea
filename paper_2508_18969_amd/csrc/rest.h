// Which cells of a fused network's batch run layer by layer: the rest that whole
// rounds of the fused kernel's tiles leave, where it is small.  (Plain C++.)
#pragma once
#include <stdint.h>

namespace chemdnn {

// The most such cells on a device of n_cu compute units, of `cells` measured (and
// provided for) on 256.  A fused tile takes the same time on any device, the
// layer kernels split a layer over the compute units: with fewer of them the
// layer kernels break even at proportionally fewer cells.  Whole cell-blocks.
inline int64_t rest_limit(int64_t cells, int n_cu) {
  return n_cu < 256 ? cells * n_cu / 256 / 16 * 16 : cells;
}

// Cells at the end of a batch of n that run layer by layer, for rounds of
// `round` cells.  Behind whole rounds the layer kernels have to wait for the
// last fused tile, while a fused rest starts on the compute units that are done:
// there the limit is lower (2/3 in FP32, half in 16 bits): of
// 31-1600-800-400-29, 16,384 + 2,048 cells in FP16 take 101 us fused and 95 in two
// parts, 16,384 + 3,627 take 102 and 103; 8,192 + 4,008 cells in FP32 419 and 366.
inline int64_t rest_cells(int64_t n, int64_t round, int64_t limit, bool fp32) {
  const int64_t rest = n % round;
  if (n >= round) limit = fp32 ? limit * 2 / 3 : limit / 2;
  return rest <= limit ? rest : 0;
}

}  // namespace chemdnn
