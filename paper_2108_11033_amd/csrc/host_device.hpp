// Functions that kernels and host code (also a plain C++ build of it, for host-side checks) share.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define GRIM_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define GRIM_HOST_DEVICE inline
#endif
