// The instances of the pair kernel (dh_pairs.h) for one precision and one
// accumulation mode: compiled once per DH_REAL (float, double) and DH_MODE
// (HistMode), side by side.
#include "dh_pairs.h"

namespace dh {

template <>
PairFn pick_pairs<DH_REAL, DH_MODE>(int r, int box) {
  return r == 8 ? pick_box<DH_REAL, 8, DH_MODE>(box) : pick_box<DH_REAL, 4, DH_MODE>(box);
}

}  // namespace dh
