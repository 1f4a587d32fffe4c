// Half-precision mode with the k loop cut into parts (skinny problems): the parts cannot add to
// an f16 C -- that would round once per part -- so they add, atomically and in f32, to a
// workspace of M x N floats that starts at zero, and a second pass adds the workspace to C with
// the mode's one rounding to nearest even.  This file holds the two small passes around the
// GEMM launch (zero the workspace; C = round(C + workspace)).
#include "gemm_device.h"
#include "../../include/gemm_f16.h"

namespace {

using namespace gemm_dev;

__global__ __launch_bounds__(256) void splitk_zero_kernel(float* __restrict__ ws, int64_t n4)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n4) reinterpret_cast<floatx4*>(ws)[i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
}

// Four columns a thread, by 32-bit indexes: N is a multiple of 8 where the k loop is cut, and C is only known to be 2-byte
// aligned.  Bound by its launch and one trip to memory, 8 MB for 2^20 results.  (An element a thread, with a
// 64-bit division each: the three launches of (256,4096,16384) 64.2 -> 62.2 us, (128,8192,8192) 49.5 -> 47.6,
// (48,16384,4096) 43.2 -> 42.4, (12,1032,8200) 13.1 -> 12.8.)
typedef half_t half4_any __attribute__((ext_vector_type(4), aligned(2)));
__global__ __launch_bounds__(256) void splitk_finish_f16_kernel(const float* __restrict__ ws, half_t* __restrict__ C, int64_t ldc, uint32_t n4, uint32_t per_row)
{
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const uint32_t r = i / per_row, c = 4 * (i - r * per_row);
    half4_any* const p = reinterpret_cast<half4_any*>(C + (int64_t)r * ldc + c);
    const floatx4 s = reinterpret_cast<const floatx4*>(ws)[i];
    const half4_any v = *p;
    half4_any o;
#pragma unroll
    for (int e = 0; e < 4; e++) o[e] = (half_t)((float)v[e] + s[e]);   // exact widening, f32 addition, one rounding to nearest even
    *p = o;
}

// The library's own scratch memory for gemm_f16_f16acc_static_workspace: 2^20 floats (4 MB) per
// GPU the library runs on, held until the process ends; it covers every problem that the
// workspace form cuts along k.  The name below is a host-side stand-in, not a device address:
// host code uses the pointer that static_scratch() hands out.
constexpr int64_t STATIC_SCRATCH_FLOATS = 1 << 20;
static __device__ __align__(256) float scratch[STATIC_SCRATCH_FLOATS];

constexpr int MAX_DEVICES = 64;
float* g_scratch_ptr[MAX_DEVICES] = {};

}  // namespace

// The current device's copy of the scratch array (its address is asked for once per device, with
// that device current) and its size in floats.
int splitk_f16_static_scratch(float** ptr, int64_t* floats)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return GEMM_F16_ERR_LAUNCH;
    if (!g_scratch_ptr[dev]) {
        float* p = nullptr;
        if (hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GEMM_F16_ERR_LAUNCH;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    *floats = STATIC_SCRATCH_FLOATS;
    return GEMM_F16_OK;
}

// n floats (a multiple of 4, 16-byte aligned) to zero
int splitk_f16_zero(float* ws, int64_t n, hipStream_t stream)
{
    const int64_t n4 = n / 4, blocks = (n4 + 255) / 256;
    if (blocks > INT32_MAX) return GEMM_F16_ERR_SIZE;
    if (blocks > 0) hipLaunchKernelGGL(splitk_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, ws, n4);
    return hipGetLastError() == hipSuccess ? GEMM_F16_OK : GEMM_F16_ERR_LAUNCH;
}

// C (f16, M x N, pitch ldc) = round(C + ws (f32, M x N, pitch N)); N a multiple of 4
int splitk_f16_finish(const float* ws, void* C, int64_t ldc, int64_t M, int64_t N, hipStream_t stream)
{
    const int64_t n4 = M * N / 4;
    if (n4 > INT32_MAX) return GEMM_F16_ERR_SIZE;
    if (n4 > 0) hipLaunchKernelGGL(splitk_finish_f16_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream, ws, (half_t*)C, ldc, (uint32_t)n4, (uint32_t)(N / 4));
    return hipGetLastError() == hipSuccess ? GEMM_F16_OK : GEMM_F16_ERR_LAUNCH;
}
