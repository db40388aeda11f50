// Enough of a HIP runtime to compile the matrix-core transforms (fm_mat.hip)
// for the host, where lanes.h runs their wavefronts in lockstep.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

#define __global__
#define __device__
#define __host__
#define __shared__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

// (the names the real headers give these types in the launchers' signatures)
template <typename T, unsigned n> struct HIP_vector_type;
template <> struct HIP_vector_type<int, 2> { int x, y; };
typedef HIP_vector_type<int, 2> int2;
typedef struct ihipStream_t* hipStream_t;
enum hipError_t { hipSuccess = 0 };
enum { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline int64_t min(int64_t a, int64_t b) { return a < b ? a : b; }
inline int64_t max(int64_t a, int64_t b) { return a > b ? a : b; }

#include "../lanes.h"

#define threadIdx lanes::thread_idx
#define blockIdx lanes::block_idx
#define blockDim lanes::block_dim
#define __syncthreads lanes::barrier
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, x, y, z) lanes::mfma<float>(a, b, c)
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, x, y, z) lanes::mfma<double>(a, b, c)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define hipFuncSetAttribute(...) hipSuccess
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
  lanes::launch(grid, block, lds, [&] { kernel(__VA_ARGS__); })
