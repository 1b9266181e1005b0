// One matrix-core instruction per wavefront on given operands, for the tests of what the library assumes about their
// roundings (operand and result layouts as its kernels use them).
#include <hip/hip_runtime.h>

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// d[n][32][32] = a[n][32][16] b[n][32][16]^T + c[n][32][32]
__global__ __launch_bounds__(64) void k_f16(const half8 *a, const half8 *b, const float *c, float *d)
{
    const int lane = threadIdx.x, l31 = lane & 31, half = lane >> 5;
    const size_t m = blockIdx.x;
    floatx16 acc;
    for (int i = 0; i < 16; ++i) acc[i] = c[m * 1024 + ((i & 3) + 8 * (i >> 2) + 4 * half) * 32 + l31];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[m * 64 + l31 * 2 + half], b[m * 64 + l31 * 2 + half], acc, 0, 0, 0);
    for (int i = 0; i < 16; ++i) d[m * 1024 + ((i & 3) + 8 * (i >> 2) + 4 * half) * 32 + l31] = acc[i];
}

// d = a[n][32][2] b[n][32][2]^T + c
__global__ __launch_bounds__(64) void k_f32(const float *a, const float *b, const float *c, float *d)
{
    const int lane = threadIdx.x, l31 = lane & 31, half = lane >> 5;
    const size_t m = blockIdx.x;
    floatx16 acc;
    for (int i = 0; i < 16; ++i) acc[i] = c[m * 1024 + ((i & 3) + 8 * (i >> 2) + 4 * half) * 32 + l31];
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[m * 64 + l31 * 2 + half], b[m * 64 + l31 * 2 + half], acc, 0, 0, 0);
    for (int i = 0; i < 16; ++i) d[m * 1024 + ((i & 3) + 8 * (i >> 2) + 4 * half) * 32 + l31] = acc[i];
}

extern "C" int probe_f16(const void *a, const void *b, const float *c, float *d, int n, hipStream_t s)
{
    if (n <= 0) return 1;
    hipLaunchKernelGGL(k_f16, dim3(n), dim3(64), 0, s, (const half8 *)a, (const half8 *)b, c, d);
    return hipGetLastError() != hipSuccess;
}
extern "C" int probe_f32(const float *a, const float *b, const float *c, float *d, int n, hipStream_t s)
{
    if (n <= 0) return 1;
    hipLaunchKernelGGL(k_f32, dim3(n), dim3(64), 0, s, a, b, c, d);
    return hipGetLastError() != hipSuccess;
}
