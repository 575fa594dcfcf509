// grad_x2 of the product with x2 shared by the channels of an edge, from the edge's Gram matrix:
//   gx2[n][k2] = sum_{k1, k3} T[k1][k2][k3] G[k1][k3],   G[k1][k3] = sum_c x1[n][c][k1] g[n][c][k3].
// The sum over the channels comes first, as a matrix product on v_mfma_f32_16x16x4f32 (full fp32:
// its products and sums are those of FMAs), so the tensor is contracted once per edge and not once
// per channel, and no per-channel rows go through memory.
//
// One wave per edge: its G is NT x NT tiles in accumulators, both operands come straight from
// global memory (a lane reads NT neighbouring columns of row lane / 16, one load in fp32),
// 4 kStep channels at a time.  Then the workgroup's 4 G lie in LDS and its 256 threads run
// the tensor's entries over them: an entry is loaded once for 4 edges.
//
// Bound by the reading of x1 and grad_out: L = 3, fp32, 8,192 edges x 100 channels 220 -> 69 us
// (the per-channel products into a workspace and their sum before), 4.6 TB/s; with one load per
// column in place of one per lane 101 us; the fp32 matrix products alone would take 24.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_common.h"
#include "internal.h"

namespace spingtp {
namespace {

__device__ __forceinline__ void narrow(float v, float* p) { *p = v; }
__device__ __forceinline__ void narrow(float v, uint16_t* p) { *p = f32_to_bf16(v); }

// NT neighbouring values of a row, which starts at any element: one load in fp32.
typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));
typedef float f3 __attribute__((ext_vector_type(3), aligned(4)));
template <int NT>
__device__ __forceinline__ void columns(const float* p, float (&v)[NT]) {
    if constexpr (NT == 3) {
        const f3 x = *reinterpret_cast<const f3*>(p);
        v[0] = x.x, v[1] = x.y, v[2] = x.z;
    } else if constexpr (NT == 2) {
        const f2 x = *reinterpret_cast<const f2*>(p);
        v[0] = x.x, v[1] = x.y;
    } else {
        v[0] = p[0];
    }
}
template <int NT>
__device__ __forceinline__ void columns(const uint16_t* p, float (&v)[NT]) {
#pragma unroll
    for (int i = 0; i < NT; ++i) v[i] = bf16_to_f32(p[i]);
}

// tab: the table of build_gram_table.
template <int NT, typename TIO>
__global__ __launch_bounds__(kGramThreads, 4) void spingtp_gram_x2_kernel(const TIO* __restrict__ x1,
                                                                     const TIO* __restrict__ g,
                                                                     TIO* __restrict__ gx2, int64_t N, int64_t C,
                                                                     int nc, const uint32_t* __restrict__ tab) {
    constexpr int R = 16 * NT, GS = R * R + 1;  // one edge's G and a zero that padding items read
    constexpr int E = kGramThreads / 64;
    constexpr int kStep = 4;
    __shared__ float G[E * GS > E * kGramThreads ? E * GS : E * kGramThreads];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t n = static_cast<int64_t>(blockIdx.x) * E + wave;
    const int lr = lane & 15, lq = lane >> 4;
    if (n < N) {
        const TIO* px = x1 + n * C * nc;
        const TIO* pg = g + n * C * nc;
        v4f acc[NT][NT];
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        // the lane's NT columns of a row; the last lanes step back to stay in it
        const uint32_t at = static_cast<uint32_t>(lq * nc + (NT * lr < nc - NT ? NT * lr : nc - NT));
        auto multiply = [&](const float (&a)[NT], const float (&b)[NT]) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
        };
        int64_t c = 0;
#pragma unroll 1
        for (; c + 4 * kStep <= C; c += 4 * kStep) {
            const TIO* ra = px + c * nc;
            const TIO* rb = pg + c * nc;
            float a[kStep][NT], b[kStep][NT];
#pragma unroll
            for (int s = 0; s < kStep; ++s) {
                columns<NT>(ra + 4 * s * nc + at, a[s]);
                columns<NT>(rb + 4 * s * nc + at, b[s]);
            }
#pragma unroll
            for (int s = 0; s < kStep; ++s) multiply(a[s], b[s]);
        }
#pragma unroll 1
        for (; c < C; c += 4) {  // zeros past the last channel, which read row C - 1 instead
            const bool in = c + lq < C;
            const int64_t row = ((in ? c + lq : C - 1) - lq) * nc;
            float a[NT], b[NT];
            columns<NT>(px + row + at, a);
            columns<NT>(pg + row + at, b);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                a[i] = in ? a[i] : 0.f;
                b[i] = in ? b[i] : 0.f;
            }
            multiply(a, b);
        }
        float* Ge = G + wave * GS;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) Ge[(16 * i + 4 * lq + r) * R + 16 * j + lr] = acc[i][j][r];
        if (lane == 0) Ge[R * R] = 0.f;
    } else {  // past the last edge: its sums are not stored
        float* Ge = G + wave * GS;
        for (int i = lane; i < GS; i += 64) Ge[i] = 0.f;
    }
    __syncthreads();
    const int ipt = static_cast<int>(tab[0]);
    const uint32_t* __restrict__ items = tab + tab[1] + 2 * tid;
    float s[E];
#pragma unroll
    for (int e = 0; e < E; ++e) s[e] = 0.f;
#pragma unroll 4
    for (int i = 0; i < ipt; ++i) {
        const uint2 it = *reinterpret_cast<const uint2*>(items + 2 * kGramThreads * i);
        const float v = __uint_as_float(it.y);
#pragma unroll
        for (int e = 0; e < E; ++e) s[e] = fmaf(G[e * GS + it.x], v, s[e]);
    }
    __syncthreads();  // every entry is read before the threads' sums take the space
    float* part = G;
#pragma unroll
    for (int e = 0; e < E; ++e) part[e * kGramThreads + tid] = s[e];
    __syncthreads();
    // the threads of an output slot are consecutive: [first, last) in words 2 + k2, 3 + k2
    for (int i = tid; i < E * nc; i += kGramThreads) {
        const int e = i / nc, k = i - e * nc;
        const int64_t m = static_cast<int64_t>(blockIdx.x) * E + e;
        if (m >= N) break;
        float t = 0.f;
        for (uint32_t q = tab[2 + k]; q < tab[3 + k]; ++q) t += part[e * kGramThreads + q];
        narrow(t, gx2 + m * nc + k);
    }
}

template <int NT, typename TIO>
hipError_t launch(const void* x1, const void* g, void* gx2, int64_t N, int64_t C, int nc, const uint32_t* tab,
                  hipStream_t stream) {
    const int64_t blocks = (N + kGramThreads / 64 - 1) / (kGramThreads / 64);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((spingtp_gram_x2_kernel<NT, TIO>), dim3(static_cast<unsigned>(blocks)), dim3(kGramThreads), 0,
                       stream, static_cast<const TIO*>(x1), static_cast<const TIO*>(g), static_cast<TIO*>(gx2), N, C,
                       nc, tab);
    return hipGetLastError();
}

template <typename TIO>
hipError_t dispatch(const void* x1, const void* g, void* gx2, int64_t N, int64_t C, int nc, const uint32_t* tab,
                    hipStream_t stream) {
    switch ((nc + 15) / 16) {
        case 1: return launch<1, TIO>(x1, g, gx2, N, C, nc, tab, stream);
        case 2: return launch<2, TIO>(x1, g, gx2, N, C, nc, tab, stream);
        case 3: return launch<3, TIO>(x1, g, gx2, N, C, nc, tab, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_gram_x2(int dtype, const void* x1, const void* g, void* gx2, int64_t N, int64_t C, int nc,
                          const uint32_t* tab, hipStream_t stream) {
    return dtype == SPINGTP_FP32 ? dispatch<float>(x1, g, gx2, N, C, nc, tab, stream)
                                 : dispatch<uint16_t>(x1, g, gx2, N, C, nc, tab, stream);
}

}  // namespace spingtp
