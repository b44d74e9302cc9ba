// Solver kernels of kf_sstep.h with 2 iterations per synchronisation, for one keyframe.
#include "kf_sstep.h"

namespace kf {

// The kernel for `rows` pixels per thread; nullptr if none holds that many.
const void* sstep2_fn(int rows, bool var) {
#define KF_ROWS(R) \
  if (rows == R) return var ? reinterpret_cast<const void*>(&k_sstep<R, 2, true>) : reinterpret_cast<const void*>(&k_sstep<R, 2, false>);
  KF_SS2_ROWS(KF_ROWS)
#undef KF_ROWS
  return nullptr;
}

}  // namespace kf
