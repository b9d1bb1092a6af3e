// The device names that the line filter's headers use, as plain host code: lets a
// host compiler take those headers for the CPU tests.  A lane is a thread, and
// the lanes of a wave meet at its barrier (lane_barrier, the including program's).
#pragma once
#include <cmath>
#include <cstddef>
#include <cstdint>

using std::exp;
using std::fabs;
using std::floor;
using std::fmax;
using std::fmin;

#define __device__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() lane_barrier()
#define __builtin_amdgcn_sched_barrier(mask) ((void)0)

void lane_barrier();

struct HostIndex { int x; };
static HostIndex threadIdx{0}, blockIdx{0}, blockDim{1}, gridDim{1};

inline void __syncthreads() {}
inline int __syncthreads_or(int v) { return v; }
inline int __any(int v) { return v; }
inline unsigned long long __ballot(int v) { return v ? 1ull : 0ull; }
inline int __lane_id() { return 0; }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline int atomicOr(int *p, int v)
{
    const int old = *p;
    *p |= v;
    return old;
}

typedef int hipError_t;
typedef void *hipStream_t;
