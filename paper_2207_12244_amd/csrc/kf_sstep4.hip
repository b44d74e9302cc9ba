// Solver kernels of kf_sstep.h with 4 iterations per synchronisation, for one keyframe.
#include "kf_sstep.h"

namespace kf {

size_t sstep_smem_bytes(const Tiling& t) {
  return ss_head_bytes(t.s, t.rows) + (size_t)ss_arrays(t.rows) * t.cells * sizeof(float);
}

// The kernel for `rows` pixels per thread; nullptr if none holds that many.
const void* sstep4_fn(int rows, bool var) {
#define KF_ROWS(R) \
  if (rows == R) return var ? reinterpret_cast<const void*>(&k_sstep<R, 4, true>) : reinterpret_cast<const void*>(&k_sstep<R, 4, false>);
  KF_SS4_ROWS(KF_ROWS)
#undef KF_ROWS
  return nullptr;
}

}  // namespace kf
