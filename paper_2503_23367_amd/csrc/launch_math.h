// Index and plan arithmetic of the launches, without any HIP type: host code, kernels and a plain C++ compiler take
// the same lines, so the arithmetic can be checked at sizes that no test would launch.
#pragma once

#if defined(__HIPCC__)
#define FV_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define FV_HOST_DEVICE inline
#endif

namespace fv {

// A launch that clears arrival counters on the side (ZeroCounters) lets its first workgroups do it: thread `thread` of
// workgroup `block` clears first, first + step, ...  Grids have up to 2^31 workgroups, so the flat thread index of all of
// them does not fit 32 bits; of the first 256 it does.
constexpr unsigned kClearBlocks = 256;
constexpr unsigned kClearThreads = 256;   // threads of such a workgroup
struct CounterShare {
    int first, step;
};
FV_HOST_DEVICE bool clears_counters(unsigned block) { return block < kClearBlocks; }
FV_HOST_DEVICE CounterShare counter_share(unsigned block, unsigned thread, unsigned blocks) {
    const unsigned used = blocks < kClearBlocks ? blocks : kClearBlocks;
    return {(int)(block * kClearThreads + thread), (int)(used * kClearThreads)};
}

}  // namespace fv
