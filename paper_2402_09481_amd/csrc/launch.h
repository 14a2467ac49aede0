// Launching a kernel on a stream, or adding it to the graph that this thread records.
#pragma once
#include <tuple>
#include <type_traits>
#include <utility>

#include <hip/hip_ext.h>

#include "kernels.h"

namespace ext {

// An event that one launch of a sequence completes by itself, as part of the kernel's
// own dispatch: a record behind the kernel is a packet of its own and kept the next
// call's first kernel waiting 2.9 us (13.4 -> 16.3 us a call of three short kernels,
// 13.4 with the event on the last of them).
struct LaunchEvent {
    hipEvent_t ev = nullptr;
    bool recorded = false;  // a launch has carried it
};
// Arms le (may be null) for the next launch of this thread.
void set_launch_event(LaunchEvent *le);

extern thread_local GraphRecorder *t_graph_recorder;
extern thread_local LaunchEvent *t_launch_event;

// Launches kern on stream s, or adds it to the recording graph of this thread.
// The arguments are converted to the kernel's parameter types first; both paths
// pass pointers to those values (a graph node copies them when it is added). An armed
// launch event goes with the launch.
template <typename... P, typename... A>
static hipError_t launch_k(void (*kern)(P...), dim3 grid, dim3 block, size_t shmem, hipStream_t s, A &&...args) {
    static_assert(sizeof...(P) == sizeof...(A), "argument count");
    std::tuple<std::decay_t<P>...> vals(std::forward<A>(args)...);
    void *ptrs[sizeof...(P) > 0 ? sizeof...(P) : 1];
    std::apply([&](auto &...v) {
        int i = 0;
        ((ptrs[i++] = (void *)&v), ...);
    }, vals);
    if (GraphRecorder *r = t_graph_recorder) {
        if (r->err != hipSuccess) return r->err;
        hipKernelNodeParams kp = {};
        kp.func = (void *)kern;
        kp.gridDim = grid;
        kp.blockDim = block;
        kp.sharedMemBytes = (unsigned)shmem;
        kp.kernelParams = ptrs;
        kp.extra = nullptr;
        hipGraphNode_t node = nullptr;
        r->err = hipGraphAddKernelNode(&node, r->graph, r->last ? &r->last : nullptr, r->last ? 1 : 0, &kp);
        if (r->err == hipSuccess) r->last = node;
        return r->err;
    }
    if (LaunchEvent *le = t_launch_event) {
        t_launch_event = nullptr;
        const hipError_t e = hipExtLaunchKernel((const void *)kern, grid, block, ptrs, shmem, s, nullptr, le->ev, 0);
        le->recorded = e == hipSuccess;
        return e;
    }
    return hipLaunchKernel((const void *)kern, grid, block, ptrs, shmem, s);
}

}  // namespace ext
