// Host stand-in for the HIP runtime header: what csrc/kernels.h and csrc/gf2.h name,
// so that the GF(2)[t] path's host-compilable parts build as plain C++.
#pragma once
#include <stddef.h>
#include <stdint.h>
#define __device__
#define __host__
typedef int hipError_t;
typedef void *hipStream_t, *hipGraph_t, *hipGraphNode_t;
constexpr int hipSuccess = 0;
struct uint2 {
    uint32_t x, y;
};
