// Work of others that a launch takes along as extra blocks of 256 threads at the end of its grid: weights to cut, side tasks of a sampling
// call, the reduction of weight gradients.
#pragma once
#include "gemm_tile.hpp"
#include "handles.hpp"
#include "side.hpp"

namespace no {

// Extra blocks of a launch that cuts weights for products behind it, ahead of those of its side tasks.
struct PlanesSide {
    uint32_t first_block = 0, end_block = 0;      // (end_block: where the side tasks begin)
    CutJobs cut;
    SideTasks side;
};
__device__ __forceinline__ void run_side_tasks(const PlanesSide& p) {
    if (blockIdx.x < p.end_block) run_cut_jobs(p.cut, blockIdx.x - p.first_block);
    else run_side_tasks(p.side);
}
// Extra blocks that reduce the weight gradients of the launch before.
struct ReduceSide {
    uint32_t first_block = 0, blocks = 0;      // (blocks: of each product)
    ReduceArgs reduce;
};
__device__ __forceinline__ void run_side_tasks(const ReduceSide& r) {
    const uint32_t block = blockIdx.x - r.first_block;
    reduce_block(r.reduce, block % r.blocks, (int)(block / r.blocks));
}

// Calls launch(side, grid) with what rides on a launch of `own` blocks: the cut weights, side tasks, both or neither.
template <class Launch>
static void launch_with_riders(const CutJobs* cut, no_blocks_s* side_of, uint32_t own, Launch launch) {
    const uint32_t end = own + (cut ? cut->blocks() : 0u);
    SideTasks side;
    side.first_block = end;
    if (side_of) side_take(side_of, end, &side);
    const uint32_t grid = end + side.side_blocks();
    if (end > own) {
        PlanesSide p;
        p.first_block = own; p.end_block = end; p.cut = *cut; p.side = side;
        launch(p, grid);
    } else if (side.n > 0) {
        launch(side, grid);
    } else {
        NoSideTasks none;
        none.first_block = own;
        launch(none, grid);
    }
}

}  // namespace no
