// ppt_work.h -- arithmetic of the persistent kernels' work distribution (integer host/device functions, no state).
#pragma once

#ifdef __HIP__
#define PPT_HD __host__ __device__ __forceinline__
#else
#define PPT_HD inline
#endif

namespace ppt {

constexpr int WORK_SHARDS = 16, WORK_SHARDS_FEW = 4;  // (a workgroup has four wavefronts)

// Counters that `waves` wavefronts (a multiple of four) share, wavefront w taking from counter w mod that number.
// Every counter needs a wavefront that takes from it until its batches end: the batches of a counter without one
// would be left out.
PPT_HD int work_shards(int waves) { return waves < WORK_SHARDS ? WORK_SHARDS_FEW : WORK_SHARDS; }
// The batch that ticket t of a counter stands for: over all tickets and counters every batch once, and rising in t,
// so that a wavefront whose ticket lies beyond the end has seen the last of its counter.
PPT_HD int work_batch(int t, int shard, int shards) { return t * shards + ((shard + t) & (shards - 1)); }

}  // namespace ppt
