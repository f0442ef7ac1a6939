// Small grouped kernels around the Adafactor rules (the base optimizer of the
// paper's experiments, Section 3.1; unfactored variant, Section 3.3) and the end of an
// accumulation cycle (Algorithm 1: the accumulator starts each cycle at zero).
// All reductions run in a fixed order, so results are reproducible bit for bit.
#include "flora_internal.h"

namespace flora {

namespace {

__device__ __forceinline__ float block_sum_256(float v, float* lds)
{
    const int tid = threadIdx.x;
    lds[tid] = v;
    __syncthreads();
#pragma unroll
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) lds[tid] += lds[tid + s];
        __syncthreads();
    }
    const float r = lds[0];
    __syncthreads();
    return r;
}

// The same for 1024 threads: the waves' sums through lds[16], added in wave order.
__device__ __forceinline__ float block_sum_1024(float v, float* lds)
{
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) r += lds[w];
    __syncthreads();
    return r;
}

// Sum of `count` values `stride` floats apart, in order, eight loads in flight (one at a time the sums over
// 32 row blocks of one 1024 x 1024 matrix took 30 us of memory round trips).
__device__ __forceinline__ float strided_sum(const float* p, int count, long long stride)
{
    float s = 0.f;
    int c = 0;
    for (; c + 8 <= count; c += 8) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = ldg(p + (long long)(c + e) * stride);
#pragma unroll
        for (int e = 0; e < 8; ++e) s += v[e];
    }
    for (; c < count; ++c) s += ldg(p + (long long)c * stride);
    return s;
}

// R_i <- beta2 R_i + (1 - beta2) (rowmean(Gt^2) + eps1), K_j likewise by column,
// scal[0] <- mean(R), scal[1] <- 1 (no clipping until rms_finalize says otherwise).
__global__ __launch_bounds__(1024) void stats_finalize_kernel(const MatDev* __restrict__ mats,
                                                              float beta2, float eps1)
{
    __shared__ float lds[16];
    const MatDev& M = mats[blockIdx.x];
    const long long n = M.n, m = M.m;
    const int tid = threadIdx.x;
    float rsum = 0.f;
    for (long long i = tid; i < n; i += 1024) {
        const float s = strided_sum(M.rowpart + i, M.ncolchunks, n);
        const float r = beta2 * M.row_stat[i] + (1.f - beta2) * (s / (float)m + eps1);
        M.row_stat[i] = r;
        rsum += r;
    }
    for (long long j = tid; j < m; j += 1024) {
        const float s = strided_sum(M.colpart + j, M.nrowblocks, m);
        M.col_stat[j] = beta2 * M.col_stat[j] + (1.f - beta2) * (s / (float)n + eps1);
    }
    const float tot = block_sum_1024(rsum, lds);
    if (tid == 0) {
        M.scal[0] = tot / (float)n;
        M.scal[1] = 1.f;
    }
}

// scal[1] <- 1 / max(1, RMS(U) / clip_d), RMS(U)^2 = sum of the workgroup partials / (n m)
// (1 when clip_d == 0: no clipping);  scal[2] <- max(eps2, RMS(W)) from the caller's sum of W^2
// when the step is relative to the parameter scale, else 1.
// (gram: the partial sums of U^2 are those of the quadratic-form pass, one per row block)
__global__ __launch_bounds__(256) void rms_finalize_kernel(const MatDev* __restrict__ mats, float clip_d,
                                                           int scale_parameter, float eps2, int gram)
{
    __shared__ float lds[256];
    const MatDev& M = mats[blockIdx.x];
    const int tid = threadIdx.x;
    float tot = 0.f;
    if (gram) {
        // mean(R) from the row blocks' sums of the new R, which the quadratic-form pass left in rowpart
        float s = 0.f;
        for (int i = tid; i < M.item0; i += 256) s += M.rowpart[i];
        const float mean_r = block_sum_256(s, lds) / (float)M.n;
        __syncthreads();
        if (tid == 0) { M.scal[0] = mean_r; M.scal[1] = 1.f; }
        tot = mean_r;                                      // the factor the clipping partials still lack
    }
    if (clip_d > 0.f) {
        float s = 0.f;
        const int np = gram ? M.item0 : M.nitems;
        for (int i = tid; i < np; i += 256) s += M.itempart[i];
        tot = block_sum_256(s, lds) * (gram ? tot : 1.f);
    }
    if (tid == 0) {
        float clip = 1.f;
        if (clip_d > 0.f) {
            const float rms = sqrtf(tot / ((float)M.n * (float)M.m));
            const float d = rms / clip_d;
            clip = 1.f / (d > 1.f ? d : 1.f);
        }
        M.scal[1] = clip;
        float ps = 1.f;
        if (scale_parameter) {
            const float rmsw = sqrtf(M.wsumsq[0] / ((float)M.n * (float)M.m));
            ps = rmsw > eps2 ? rmsw : eps2;
        }
        M.scal[2] = ps;
    }
}

// wsumsq <- sum of the update pass's per-workgroup partial sums of the new W^2
__global__ __launch_bounds__(256) void wsumsq_finalize_kernel(const MatDev* __restrict__ mats)
{
    __shared__ float lds[256];
    const MatDev& M = mats[blockIdx.x];
    if (!M.wsumsq) return;
    const int tid = threadIdx.x;
    float s = 0.f;
    for (int i = tid; i < M.nitems; i += 256) s += M.itempart[i];
    const float tot = block_sum_256(s, lds);
    if (tid == 0) M.wsumsq[0] = tot;
}

// Sum of W^2 from scratch: workgroup b of matrix l sums the float4s b, b + 256, ... of W
// (and the last n m % 4 values in workgroup 0) into partials[l][b].
template <typename WT>
__global__ __launch_bounds__(256) void weight_sumsq_kernel(const MatDev* __restrict__ mats,
                                                           float* __restrict__ partials)
{
    __shared__ float lds[256];
    const MatDev& M = mats[blockIdx.y];
    const long long total = M.n * M.m, total4 = total >> 2;
    const WT* W = reinterpret_cast<const WT*>(M.weight);
    const int tid = threadIdx.x;
    float s = 0.f;
    for (long long i = (long long)blockIdx.x * 256 + tid; i < total4; i += (long long)kSumsqBlocks * 256) {
        v4f w;
        if (sizeof(WT) == 4) {
            w = ldg4(reinterpret_cast<const float*>(W) + 4 * i);
        } else {
            const v2u pk = ldg2(reinterpret_cast<const uint16_t*>(W) + 4 * i);
            w = v4f{bf16_bits_to_f32(pk.x & 0xffffu), bf16_bits_to_f32(pk.x >> 16),
                    bf16_bits_to_f32(pk.y & 0xffffu), bf16_bits_to_f32(pk.y >> 16)};
        }
        s = __builtin_fmaf(w.x, w.x, s);
        s = __builtin_fmaf(w.y, w.y, s);
        s = __builtin_fmaf(w.z, w.z, s);
        s = __builtin_fmaf(w.w, w.w, s);
    }
    if (blockIdx.x == 0 && tid < (int)(total & 3)) {
        const float w = load_elem(W + 4 * total4 + tid);
        s = __builtin_fmaf(w, w, s);
    }
    const float tot = block_sum_256(s, lds);
    if (tid == 0) partials[(long long)blockIdx.y * kSumsqBlocks + blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void weight_sumsq_finalize_kernel(const MatDev* __restrict__ mats,
                                                                    const float* __restrict__ partials)
{
    __shared__ float lds[256];
    const MatDev& M = mats[blockIdx.x];
    const float tot = block_sum_256(partials[(long long)blockIdx.x * kSumsqBlocks + threadIdx.x], lds);
    if (threadIdx.x == 0) M.wsumsq[0] = tot;
}

// A descriptor image from pinned host memory into device memory, `gen` into *done (pinned) once it has been
// read.  A copy engine's transfer of the same few KB sits between two kernels of the stream with a
// queue-to-queue dependency on either side: compress calls on 96 matrices with pointers not seen before
// 28.9 us each as a copy and an event, 12.0 with this kernel (8.2 with pointers seen before); on one
// matrix 13.8 and 10.3 (7.5).
__global__ __launch_bounds__(1024) void upload_image_kernel(const v4u* src, v4u* __restrict__ dst, int n16, uint32_t* done, uint32_t gen)
{
    for (int i = threadIdx.x; i < n16; i += 4 * 1024) {
        v4u v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = i + 1024 * e < n16 ? src[i + 1024 * e] : v4u{0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + 1024 * e < n16) dst[i + 1024 * e] = v[e];
    }
    __syncthreads();                           // every thread's reads have returned (their values were stored)
    if (threadIdx.x == 0) __hip_atomic_store(done, gen, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void zero_state_kernel(const MatDev* __restrict__ mats, int r)
{
    const MatDev& M = mats[blockIdx.y];
    const long long total4 = (M.n * r) >> 2;   // r is a multiple of 4
    float4* p = reinterpret_cast<float4*>(M.state);
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total4; i += (long long)gridDim.x * 256)
        p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

}  // namespace

hipError_t launch_stats_finalize(const MatDev* mats, int count, float beta2, float eps1, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(stats_finalize_kernel, dim3((unsigned)count), dim3(1024), 0, s, mats, beta2, eps1);
    return hipGetLastError();
}

hipError_t launch_rms_finalize(const MatDev* mats, int count, float clip_d, int scale_parameter, float eps2, int gram,
                               hipStream_t s)
{
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(rms_finalize_kernel, dim3((unsigned)count), dim3(256), 0, s, mats, clip_d,
                       scale_parameter, eps2, gram);
    return hipGetLastError();
}

hipError_t launch_wsumsq_finalize(const MatDev* mats, int count, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(wsumsq_finalize_kernel, dim3((unsigned)count), dim3(256), 0, s, mats);
    return hipGetLastError();
}

hipError_t launch_weight_sumsq(const MatDev* mats, int count, int weight_is_bf16, float* partials, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    static_assert(kSumsqBlocks == 256, "one partial per thread of the finalize kernel");
    if (weight_is_bf16)
        hipLaunchKernelGGL(weight_sumsq_kernel<uint16_t>, dim3(kSumsqBlocks, (unsigned)count), dim3(256), 0, s, mats, partials);
    else
        hipLaunchKernelGGL(weight_sumsq_kernel<float>, dim3(kSumsqBlocks, (unsigned)count), dim3(256), 0, s, mats, partials);
    hipLaunchKernelGGL(weight_sumsq_finalize_kernel, dim3((unsigned)count), dim3(256), 0, s, mats, partials);
    return hipGetLastError();
}

hipError_t launch_upload_image(const void* src, void* dst, size_t bytes, uint32_t* done, uint32_t gen, hipStream_t s)
{
    hipLaunchKernelGGL(upload_image_kernel, dim3(1), dim3(1024), 0, s, static_cast<const v4u*>(src), static_cast<v4u*>(dst),
                       (int)(bytes / 16), done, gen);
    return hipGetLastError();
}

hipError_t launch_zero_state(const MatDev* mats, int count, int r, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_state_kernel, dim3(16, (unsigned)count), dim3(256), 0, s, mats, r);
    return hipGetLastError();
}

}  // namespace flora
