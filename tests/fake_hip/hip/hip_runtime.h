// The few HIP names that the memory pool uses, for a build without a GPU; pool_check.cpp
// defines them.
#pragma once
#include <cstddef>
#include <cstdint>
typedef enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 } hipError_t;
typedef struct FakeStream *hipStream_t;
struct hipFuncAttributes;
hipError_t hipMalloc(void **p, size_t bytes);
hipError_t hipFree(void *p);
hipError_t hipGetDevice(int *dev);
hipError_t hipDeviceSynchronize();
hipError_t hipGetLastError();
