// Host-side launchers of the device kernels (kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace sepso {

void launch_geom(const Pools& pl, int n_inst, int move, hipStream_t s);
void launch_philox(uint32_t first, uint32_t c1, uint32_t c2, uint32_t c3, uint64_t key, int64_t n,
                   uint32_t* out, hipStream_t s);
void launch_init(const Pools& pl, int n_blocks, int frame_override, int use_prev, hipStream_t s);
bool step_supported(int K);
// 32-bit words of dynamic LDS the fused iteration takes per block.
size_t iter_lds_words(int pos_floats, int stage_floats, int gb_floats, int ngb_max, int ppb_max,
                      int threads);
size_t iter_lds_bytes(const Pools& pl, int threads);
// One iteration's tile kernel (fused, or the update alone without
// STEP_FIT) over n_blocks entries of pl.blk_tiles; false for an unsupported K.
bool launch_tiles(const Pools& pl, int K, int n_blocks, int threads, int flags, hipStream_t s);
// Launch `it` (0 ..) of a frame whose iterations find the bests at their start; false for a K it is not built for.
bool launch_one(const Pools& pl, int K, int n_blocks, int threads, int it, hipStream_t s);
// Between launches `it` and it + 1 of such a frame, where an online outer step may be due.
void launch_hsef_one(const Pools& pl, int it, hipStream_t s);
// All iterations (at most iters) of the current frame of every instance, one
// workgroup each; false for a K it is not built for.
struct FrameLaunch {
  int block = 0;      // threads of one block of ppb particles (a tile's over its wave groups)
  int threads = 0;    // whole blocks
  int ahead = 1;      // iterations whose random factors are drawn together (threads per particle at most)
  bool one = false;   // every instance's blocks, and a thread per particle, fit at once
  size_t lds = 0;     // dynamic LDS, the largest instance's
};
bool launch_frame(const Pools& pl, int K, const FrameLaunch& f, int n_inst, int iters, hipStream_t s);
size_t frame_lds_bytes(int G, int N, int W, int threads, int ahead);
// The per-instance reduce that follows the tile kernels of an iteration.
void launch_reduce(const Pools& pl, int flags, hipStream_t s);
void launch_evolve_init(const EvolveDev& ev, const Pools& pl, hipStream_t s);
void launch_evolve_step(const EvolveDev& ev, const Pools& pl, int injected, hipStream_t s);

}  // namespace sepso
