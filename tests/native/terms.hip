// csrc/terms.h on its own, for tests/test_gpu_terms.py
#include <hip/hip_runtime.h>
#include "terms.h"

// pair i: what is left of x[i] and y[i] when their top halves are taken off
__global__ void less_terms(const float *x, const float *y, float *rx, float *ry, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const tdt::MinusOne minus;
    const unsigned o = tdt::top_halves(x[i], y[i]);
    rx[i] = tdt::less_term(o, minus.low, x[i]);
    ry[i] = tdt::less_term(o, minus.high, y[i]);
}

extern "C" int run_less_terms(const float *x, const float *y, float *rx, float *ry, int n, void *stream)
{
    hipLaunchKernelGGL(less_terms, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream), x, y, rx, ry, n);
    return (int)hipGetLastError();
}
