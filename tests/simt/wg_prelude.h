// What batch.hip and tc_reduce.hip use beyond the graph and job sweeps, for
// the CPU emulation (test infrastructure only; see hip/hip_runtime.h).  Their
// dynamic LDS, `extern __shared__`, is SIMT_DYNAMIC after wg_build.py: one plain
// array per source.
#pragma once
#include "hip/hip_runtime.h"

#define SIMT_DYNAMIC extern
struct ulonglong2 { unsigned long long x, y; };

#define __builtin_amdgcn_readfirstlane(v) ((int)__shfl((int)(v), 0))
#define __builtin_amdgcn_readlane(v, l) ((int)__shfl((int)(v), (l)))
static inline unsigned simt_add_sat(unsigned a, unsigned b) { return a + b < a ? ~0u : a + b; }
#define __builtin_elementwise_add_sat(a, b) simt_add_sat((a), (b))
static int simt_or_flag = 0;
__attribute__((noinline)) static int __syncthreads_or(int p) {
    __syncthreads();
    simt_or_flag = 0;
    __syncthreads();
    if (p) simt_or_flag = 1;
    __syncthreads();
    return simt_or_flag;
}

#define HIP_SYMBOL(x) ((void*)(x))
static inline hipError_t hipGetSymbolAddress(void** p, void* s) { *p = s; return 0; }
enum { hipFuncAttributeMaxDynamicSharedMemorySize = 0, hipStreamNonBlocking = 1, hipStreamCaptureModeThreadLocal = 1 };
static inline hipError_t hipFuncSetAttribute(const void*, int, int) { return 0; }
static inline hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorInvalidValue; }
static inline hipError_t hipStreamDestroy(hipStream_t) { return 0; }
static inline hipError_t hipStreamBeginCapture(hipStream_t, int) { return hipErrorInvalidValue; }
static inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorInvalidValue; }
static inline hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, void*, char*, size_t) { return hipErrorInvalidValue; }
static inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorInvalidValue; }
static inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return 0; }
static inline hipError_t hipGraphDestroy(hipGraph_t) { return 0; }
