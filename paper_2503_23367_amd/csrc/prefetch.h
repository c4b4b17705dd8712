// Weights that a later product of the call reads, brought into the memory-side cache by workgroups of a launch that leaves CUs
// idle.  A product of a few hundred rows waits for its weights: a CU pulls in about 37 bytes a nanosecond of what comes
// from memory and more of what the cache behind the L2s holds.  With the weights there a product alone takes (us, from memory / from the
// cache) 256 x 2048 x 8192 20 / 15.5, 576 x 2048 x 8192 30 / 25; inside eight blocks FC2 of 256 rows takes 18.1.  The launch
// that fetches pays for it (24x24 25.5 -> 29.0 us, 18.2 -> 19.9 in a sub-layer step).  Half of a matrix is worth nothing to the tiled products,
// whose slowest workgroups set the time, so they are fetched whole or not at all.
#pragma once

#include "common.h"

namespace fv {

struct Prefetch {
    static constexpr int kRanges = 3;
    const char* p[kRanges] = {};
    int lines[kRanges] = {};   // of 128 bytes, inside the tensor
    int blocks = 0;            // workgroups that do it, behind the launch's own
};

// Workgroup `block` of f.blocks: a touch of four bytes brings in a line; a lane has eight touches in flight.
__device__ __forceinline__ void prefetch_lines(const Prefetch& f, int block) {
    const int step = f.blocks * (int)blockDim.x, first = block * (int)blockDim.x + (int)threadIdx.x;
#pragma unroll
    for (int r = 0; r < Prefetch::kRanges; ++r) {
        const char* const base = f.p[r];
        const int n = f.lines[r];
        for (int i = first; i < n; i += 8 * step) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = *reinterpret_cast<const uint32_t*>(base + (size_t)min(i + u * step, n - 1) * 128);
#pragma unroll
            for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(v[u]));
        }
    }
}

}  // namespace fv
