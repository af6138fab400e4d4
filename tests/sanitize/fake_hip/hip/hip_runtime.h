// The few HIP calls that the block pool makes, on host memory with a capacity
// per device, for its checks without a GPU (pool_checks.cpp defines them).
#pragma once
#include <stddef.h>

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2 };
enum { hipHostMallocCoherent = 0x40000000 };
hipError_t hipMalloc(void **p, size_t bytes);
hipError_t hipFree(void *p);
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned flags);
hipError_t hipHostFree(void *p);
hipError_t hipGetDevice(int *device);
hipError_t hipSetDevice(int device);
hipError_t hipGetLastError();
