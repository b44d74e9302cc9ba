// Solver kernel of kf_sstep.h for a batch.
#include "kf_sstep.h"

namespace kf {

namespace {

// Queues of (keyframe, member) entries as in k_solve_batch. Each entry runs the
// code that solves its keyframe alone, picked by its tiling, so a launch takes
// members of every s and strip length (in one body with the length as a bound,
// the arrays of a strip would leave the registers). Called, not inlined: one
// function of all of them spills the scalars of each. One workgroup per compute
// unit; the call saves ~900 bytes of registers per lane to scratch, once per entry.
// Members with automatic tiles, ms per batched solve against k_solve_batch with the
// same members' automatic 512-thread tiles: 16 of 160 x 120 1.87, 2.04; 4 each of
// 160 x 120 to 640 x 480 3.87, 5.08; 6 of 640 x 480 2.23, 2.42; 32 of 320 x 240
// (140 tiles, so one team at a time) 8.49, 8.20.
template <int R, int S, bool VAR>
__device__ __attribute__((noinline)) void member(const SolveArgs* tab, int ent) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint64_t p = reinterpret_cast<uint64_t>(tab);   // uniform, as the compiler cannot know of an argument
  const uint64_t q = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
  ent = __builtin_amdgcn_readfirstlane(ent);
  const auto* constant = (const __attribute__((address_space(4))) char*)q;   // scalar loads
  SolveArgs a;
  __builtin_memcpy(&a, (const void*)(constant + (size_t)(ent >> 8) * sizeof(SolveArgs)), sizeof(SolveArgs));
  sstep_member<R, S, VAR>(a, ent & 255, smem);
}

template <bool VAR>
__global__ __launch_bounds__(SS_NT) void k_sstep_batch(const SolveArgs* __restrict__ tab,
                                                       const int32_t* __restrict__ queue,
                                                       const int32_t* __restrict__ qoff) {
  const int q1 = qoff[blockIdx.x + 1];
  for (int q = qoff[blockIdx.x]; q < q1; ++q) {
    const int32_t ent = queue[q];
    const SolveArgs& a = tab[ent >> 8];
    __syncthreads();   // the previous member's last LDS reads are done
    if (a.s == 4) {
      switch (a.rows) {
#define KF_ROWS(R) case R: member<R, 4, VAR>(tab, ent); break;
        KF_SS4_ROWS(KF_ROWS)
#undef KF_ROWS
      }
    } else {
      switch (a.rows) {
#define KF_ROWS(R) case R: member<R, 2, VAR>(tab, ent); break;
        KF_SS2_ROWS(KF_ROWS)
#undef KF_ROWS
      }
    }
  }
}

}  // namespace

const void* sstep_batch_fn(bool var) {
  return var ? reinterpret_cast<const void*>(&k_sstep_batch<true>) : reinterpret_cast<const void*>(&k_sstep_batch<false>);
}

}  // namespace kf
