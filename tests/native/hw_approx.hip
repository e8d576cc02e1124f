// How far gfx950's v_rcp_f32 and v_sqrt_f32 are from the correctly rounded reciprocal and
// square root, over every operand for which the kernels rely on it being at most one bit
// pattern (tests/test_gpu_hw_approx.py):
//   v_rcp_f32   all 2^23 significands at each exponent from -49 to 102, the denominators of
//               the BF16 commit's bracketed step;
//   v_sqrt_f32  every binary32 number from 2^-96 up to infinity.
// Prints for each: operands, how many results are one pattern low, one high, and further off.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

typedef unsigned long long u64;

// Operands first + k, k < n, of which thread t takes t, t + stride, ...
template <bool Rcp>
__global__ __launch_bounds__(256) void compare(uint32_t first, uint32_t n, u64* counts) {
    u64 low = 0, high = 0, far = 0;
    for (uint64_t k = blockIdx.x * 256ull + threadIdx.x; k < n; k += gridDim.x * 256ull) {
        const float x = __uint_as_float(first + (uint32_t)k);
        const float hw = Rcp ? __builtin_amdgcn_rcpf(x) : __builtin_amdgcn_sqrtf(x);
        const float exact = Rcp ? 1.0f / x : __builtin_sqrtf(x);
        const int32_t off = (int32_t)(__float_as_uint(hw) - __float_as_uint(exact));
        low += off == -1;
        high += off == 1;
        far += off < -1 || off > 1;
    }
    atomicAdd(counts, low);
    atomicAdd(counts + 1, high);
    atomicAdd(counts + 2, far);
}

template <bool Rcp>
int run(const char* name, uint32_t first, uint32_t n, u64* counts) {
    u64 host[3] = {0, 0, 0};
    if (hipMemcpy(counts, host, sizeof host, hipMemcpyHostToDevice) != hipSuccess) return 1;
    hipLaunchKernelGGL((compare<Rcp>), dim3(4096), dim3(256), 0, 0, first, n, counts);
    if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) return 1;
    if (hipMemcpy(host, counts, sizeof host, hipMemcpyDeviceToHost) != hipSuccess) return 1;
    printf("%s %u %llu %llu %llu\n", name, n, host[0], host[1], host[2]);
    return 0;
}

int main() {
    u64* counts = nullptr;
    if (hipMalloc(&counts, 3 * sizeof(u64)) != hipSuccess) return 1;
    const uint32_t rcp_first = (uint32_t)(127 - 49) << 23, rcp_end = (uint32_t)(127 + 103) << 23;
    const uint32_t sqrt_first = (uint32_t)(127 - 96) << 23, sqrt_end = 0x7F800000u;
    const int bad = run<true>("v_rcp_f32", rcp_first, rcp_end - rcp_first, counts) |
                    run<false>("v_sqrt_f32", sqrt_first, sqrt_end - sqrt_first, counts);
    return hipFree(counts) != hipSuccess || bad;
}
