// Dtype-independent parts of the fused kernels: LDS sizing, dispatch on the
// storage type, and the counter-clearing kernel.
#include <hip/hip_runtime.h>

#include "hs_internal.h"

namespace hsk {

#define HS_DECL_GROUP(n, g)                                                                     \
    hipError_t launch_fused_##n##_g##g(int mode, int H, const TileArgs& a, int64_t nt, int grid,  \
                                       int lds, hipStream_t s);                                  \
    hipError_t launch_tiles_##n##_g##g(int H, const WalkArgs& a, int grid, hipStream_t s);
#define HS_DECL_TYPE(n) HS_DECL_GROUP(n, 0) HS_DECL_GROUP(n, 1) HS_DECL_GROUP(n, 2) HS_DECL_GROUP(n, 3)
HS_DECL_TYPE(f32)
HS_DECL_TYPE(f16)
HS_DECL_TYPE(bf16)
#define HS_DECL_STAT(g)                                                                          \
    hipError_t launch_stat_f32_g##g(int mode, int H, const TileArgs& a, int64_t nt, int grid,     \
                                    int lds, hipStream_t s);
HS_DECL_STAT(0)
HS_DECL_STAT(1)
HS_DECL_STAT(2)
HS_DECL_STAT(3)

__global__ void k_zero_i64(int64_t* p, int64_t n)
{
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        p[e] = 0;
}

int fused_lds_bytes(int T, int R, int H, int mode, int elem_bytes)
{
    (void)mode;
    return fused_stage_bytes(H, elem_bytes) + smem_tail_bytes(T, R, H);
}

#define HS_GROUP_CASES(call)                                                                    \
    switch ((H - 1) / 4) {                                                                      \
    case 0: return call(0);                                                                     \
    case 1: return call(1);                                                                     \
    case 2: return call(2);                                                                     \
    case 3: return call(3);                                                                     \
    }                                                                                           \
    return hipErrorInvalidValue;

hipError_t launch_fused(int mode, int dtype, int H, const TileArgs& a, int64_t n_tiles, int grid,
                        int lds_bytes, hipStream_t s)
{
    if (H < 1 || H > kMaxH) return hipErrorInvalidValue;
    if (mode == kModeLse) {
        if (dtype != HS_DTYPE_F32) return hipErrorInvalidValue;
#define HS_CALL(g) launch_stat_f32_g##g(mode, H, a, n_tiles, grid, lds_bytes, s)
        HS_GROUP_CASES(HS_CALL)
#undef HS_CALL
    }
    switch (dtype) {
    case HS_DTYPE_F32: {
#define HS_CALL(g) launch_fused_f32_g##g(mode, H, a, n_tiles, grid, lds_bytes, s)
        HS_GROUP_CASES(HS_CALL)
#undef HS_CALL
    }
    case HS_DTYPE_F16: {
#define HS_CALL(g) launch_fused_f16_g##g(mode, H, a, n_tiles, grid, lds_bytes, s)
        HS_GROUP_CASES(HS_CALL)
#undef HS_CALL
    }
    case HS_DTYPE_BF16: {
#define HS_CALL(g) launch_fused_bf16_g##g(mode, H, a, n_tiles, grid, lds_bytes, s)
        HS_GROUP_CASES(HS_CALL)
#undef HS_CALL
    }
    }
    return hipErrorInvalidValue;
}

hipError_t launch_tiles(int dtype, int H, const WalkArgs& a, int grid, hipStream_t s)
{
    if (H < 1 || H > kMaxH) return hipErrorInvalidValue;
    if (a.n_fops > 0) return launch_walk(dtype, H, kV, a, grid, s);   // the same strips
    switch (dtype) {
    case HS_DTYPE_F32: {
#define HS_CALL(g) launch_tiles_f32_g##g(H, a, grid, s)
        HS_GROUP_CASES(HS_CALL)
#undef HS_CALL
    }
    case HS_DTYPE_F16: {
#define HS_CALL(g) launch_tiles_f16_g##g(H, a, grid, s)
        HS_GROUP_CASES(HS_CALL)
#undef HS_CALL
    }
    case HS_DTYPE_BF16: {
#define HS_CALL(g) launch_tiles_bf16_g##g(H, a, grid, s)
        HS_GROUP_CASES(HS_CALL)
#undef HS_CALL
    }
    }
    return hipErrorInvalidValue;
}

// Streaming read of n16 16-byte words: block b sums its words (grid-stride,
// four loads in flight per thread) and writes one float, sink[b].  The
// bandwidth ceiling the detection kernels are measured against.
__global__ __launch_bounds__(256) void k_stream_read(const float4* __restrict__ p, int64_t n16,
                                                     float* __restrict__ sink)
{
    constexpr int U = 4;
    const int64_t stride = (int64_t)gridDim.x * 256;
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    float acc = 0.0f;
    for (; i + (U - 1) * stride < n16; i += U * stride) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = p[i + u * stride];
#pragma unroll
        for (int u = 0; u < U; ++u) acc += (v[u].x + v[u].y) + (v[u].z + v[u].w);
    }
    for (; i < n16; i += stride) {
        const float4 v = p[i];
        acc += (v.x + v.y) + (v.z + v.w);
    }
    __shared__ float part[4];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) sink[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

hipError_t launch_stream_read(const void* src, int64_t bytes, float* sink, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_stream_read, dim3(grid), dim3(256), 0, s, static_cast<const float4*>(src), bytes / 16,
                       sink);
    return hipGetLastError();
}

hipError_t launch_zero_i64(int64_t* p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_zero_i64, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

}  // namespace hsk
