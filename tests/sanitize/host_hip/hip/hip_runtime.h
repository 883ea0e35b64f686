// hip_runtime.h -- a host model of one workgroup, so that device headers can
// be compiled for the CPU and run under a thread sanitizer: one thread per
// lane, __syncthreads a barrier over the workgroup, a ballot a barrier over
// its wave.  Only what those headers use.
#pragma once

#include <pthread.h>
#include <stddef.h>
#include <stdint.h>

#define __device__
#define __global__
#define __forceinline__ inline
#define __builtin_amdgcn_perm host_perm
#define __builtin_amdgcn_ballot_w64 host_ballot
#define __builtin_amdgcn_fence(order, scope) ((void)0)

typedef int hipError_t;
typedef void *hipStream_t;
typedef void *hipEvent_t;

struct int2 {
    int x, y;
};
struct uint2 {
    unsigned x, y;
};
struct Index3 {
    unsigned x, y, z;
};

struct HostWave {
    pthread_barrier_t barrier;
    uint64_t votes;
};
extern thread_local Index3 threadIdx, blockIdx, blockDim, gridDim;
extern thread_local HostWave *host_wave;
extern pthread_barrier_t host_group;

inline int2 make_int2(int x, int y) { return int2{x, y}; }
inline int min(int a, int b) { return a < b ? a : b; }
inline void __syncthreads() { pthread_barrier_wait(&host_group); }
inline void atomicOr(int *p, int v) { __atomic_fetch_or(p, v, __ATOMIC_RELAXED); }

inline uint64_t host_ballot(bool p)
{
    const unsigned lane = threadIdx.x & 63;
    if (lane == 0)
        __atomic_store_n(&host_wave->votes, 0, __ATOMIC_RELAXED);
    pthread_barrier_wait(&host_wave->barrier);
    if (p)
        __atomic_fetch_or(&host_wave->votes, 1ull << lane, __ATOMIC_RELAXED);
    pthread_barrier_wait(&host_wave->barrier);
    const uint64_t v = __atomic_load_n(&host_wave->votes, __ATOMIC_RELAXED);
    pthread_barrier_wait(&host_wave->barrier);
    return v;
}

// bytes of {a, b} (b the low half) picked by the selector's bytes
inline uint32_t host_perm(uint32_t a, uint32_t b, uint32_t sel)
{
    const uint64_t both = (uint64_t)a << 32 | b;
    uint32_t r = 0;
    for (int i = 0; i < 4; ++i)
        r |= (uint32_t)(both >> (8 * ((sel >> (8 * i)) & 7)) & 0xff) << (8 * i);
    return r;
}

template <class T> inline T __shfl_xor(T v, int, int) { return v; } // not modelled
