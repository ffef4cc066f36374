// Stand-in for the HIP runtime header that lets the library's headers and host
// code compile for the CPU, for tests: the device qualifiers are empty, a wave
// is 64 fibers that meet at every cross-lane operation, and the runtime calls
// are declared (wave.h and fake_hip.h define what a test uses).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline __attribute__((always_inline))

struct uint2 {
  uint32_t x, y;
};
struct uint4 {
  uint32_t x, y, z, w;
};
inline uint2 make_uint2(uint32_t x, uint32_t y) { return uint2{x, y}; }

// ---- the lanes of a wave -----------------------------------------------------
struct LaneIndex {
  operator uint32_t() const;
};
struct ThreadIndex {
  LaneIndex x;
};
extern ThreadIndex threadIdx;

typedef uint32_t u32pair __attribute__((ext_vector_type(2)));
uint64_t __ballot(bool x);
int __builtin_amdgcn_readlane(int x, int lane);
int __builtin_amdgcn_readfirstlane(int x);
int __builtin_amdgcn_update_dpp(int old, int src, int ctrl, int row_mask, int bank_mask, bool bound_ctrl);
int __builtin_amdgcn_ds_bpermute(int addr, int x);
u32pair __builtin_amdgcn_permlane16_swap(uint32_t a, uint32_t b, bool fi, bool bc);
u32pair __builtin_amdgcn_permlane32_swap(uint32_t a, uint32_t b, bool fi, bool bc);
bool __builtin_amdgcn_inverse_ballot_w64(uint64_t m);
uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t m, uint32_t add);
uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t m, uint32_t add);
int __shfl_down(int x, int d, int width);
void __syncthreads();

inline uint32_t __builtin_amdgcn_alignbit(uint32_t hi, uint32_t lo, uint32_t s) {
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> (s & 31u));
}
inline int __popc(uint32_t x) { return __builtin_popcount(x); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }

// ---- the runtime (fake_hip.cpp) ------------------------------------------------
typedef struct ihipStream_t* hipStream_t;
typedef struct ihipEvent_t* hipEvent_t;
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
enum hipMemoryType { hipMemoryTypeUnregistered, hipMemoryTypeHost, hipMemoryTypeDevice };
enum { hipHostMallocDefault = 0, hipEventDisableSystemFence = 0 };
struct hipPointerAttribute_t {
  hipMemoryType type;
};
struct dim3 {
  uint32_t x, y, z;
  dim3(uint32_t x = 1, uint32_t y = 1, uint32_t z = 1) : x(x), y(y), z(z) {}
};
hipError_t hipLaunchKernel(const void* kernel, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t st);
hipError_t hipMalloc(void** p, size_t n);
template <class T>
hipError_t hipMalloc(T** p, size_t n) {
  return hipMalloc(reinterpret_cast<void**>(p), n);
}
hipError_t hipFree(void* p);
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags);
hipError_t hipHostFree(void* p);
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k);
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st);
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st);
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p);
hipError_t hipGetLastError();
hipError_t hipSetDevice(int d);
hipError_t hipGetDevice(int* d);
hipError_t hipDeviceSynchronize();
hipError_t hipStreamSynchronize(hipStream_t st);
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags);
hipError_t hipEventDestroy(hipEvent_t e);
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st);
hipError_t hipEventSynchronize(hipEvent_t e);
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b);
