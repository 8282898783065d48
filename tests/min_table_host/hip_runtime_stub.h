// Host stand-in for the few device built-ins that drsf_dev.h names, so that a
// workgroup's use of the table of minima can run as threads of the host
// (tests/test_min_table_host.py installs it as <hip/hip_runtime.h>).  A
// workgroup is BLOCK threads that share one barrier; the wave built-ins are
// declared only, since the table uses none.  Test infrastructure only.
#pragma once
#include <pthread.h>
#include <stdint.h>
#define __device__
#define __host__
#define __forceinline__ inline
struct StubDim { unsigned x; };
extern thread_local StubDim threadIdx;
extern StubDim blockDim;
extern pthread_barrier_t stub_barrier;
inline void __syncthreads() { pthread_barrier_wait(&stub_barrier); }
inline int32_t atomicCAS(int32_t *p, int32_t cmp, int32_t v) {
    __atomic_compare_exchange_n(p, &cmp, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
    return cmp;
}
template <class T> T atomicAdd(T *p, T v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
template <class T> T atomicExch(T *p, T v) { return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }
template <class T> T atomicMin(T *p, T v) {
    T cur = __atomic_load_n(p, __ATOMIC_SEQ_CST);
    while (v < cur && !__atomic_compare_exchange_n(p, &cur, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {}
    return cur;
}
int __lane_id();
uint64_t __ballot(int);
template <class T> T __shfl(T, int);
template <class T> T __shfl_xor(T, int);
int __popcll(unsigned long long);
int __ffsll(unsigned long long);
int __clzll(long long);
unsigned __builtin_amdgcn_mbcnt_hi(unsigned, unsigned);
unsigned __builtin_amdgcn_mbcnt_lo(unsigned, unsigned);
