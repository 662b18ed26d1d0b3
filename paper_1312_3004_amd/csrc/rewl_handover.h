// rewl_handover.h -- hand-over of blocks of 64 attempts from the wavefront that
// draws them to the one that decides them, through two records in LDS (block
// base in record handover_slot(base)).
//
// Both sides meet at the same workgroup barriers: one after block 0 is drawn,
// then one a block.  At the barrier of block i, blocks 0 .. i + 1 have been
// drawn and block i has been read, so that behind it the drawing side may
// write block i + 2 where block i was, and the deciding side reads block i + 1.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rewl_gpu {

__host__ __device__ __forceinline__ int handover_slot(int64_t base) { return (int)((base >> 6) & 1); }

// draw(base): writes the block of attempts base .. of n.
template <class Draw, class Sync>
__host__ __device__ __forceinline__ void handover_draw(int64_t n, Draw draw, Sync sync) {
    if (n > 0) draw((int64_t)0);
    sync();
    for (int64_t base = 0; base < n; base += 64) {
        if (base + 64 < n) draw(base + 64);
        sync();
    }
}

// fetch(base): reads the block; block(base): decides it, and calls
// fetch(base + 64) on the way (past the end: old words, not used).
template <class Fetch, class Sync, class Block>
__host__ __device__ __forceinline__ void handover_decide(int64_t n, Fetch fetch, Sync sync, Block block) {
    sync();
    fetch((int64_t)0);
    for (int64_t base = 0; base < n; base += 64) {
        sync();
        block(base);
    }
}

}  // namespace rewl_gpu
