// The direct kernel (forward_direct.hip) unrolled over the tensor's entries, for the spin set
// {-2..2} at L1 = L2 = Lout <= 2: out[u, o] = sum value A[u, a] B[u, b] with every index a
// compile-time constant (tensor_pattern.h).  Shared by the translation units of the bases.
//
// One lane per unit; its A, B and output rows are registers (35 + 35 + 35 used slots at degree
// 2), each product A[a] B[b] is formed once for all the outputs it enters, and the values come
// through scalar loads as the FMAs' scalar operands (the list is one sequence, read in order).
// Per 64 units that is 1,053 products and 2,003 FMAs in the paper basis and no LDS access,
// where the entry-list kernel needs two LDS gathers, two address additions, a product and an
// FMA per entry.  Rows pass through one wave-private LDS tile for coalesced 16-byte accesses.
// Measured, degree 2, 12.8 M units, fp32, paper basis: 4.58 -> 1.22 ms, 5.7 TB/s of the bytes
// it must move, so memory-bound (the arithmetic alone: 3,056 vector instructions per 64 units,
// 1.0 ms).  Bit-identical results: the entry order and the two partial sums per output are the
// entry-list kernel's.  Registers (136 at degree 2: 35 used slots of either input, two sums
// per output) end it there: degree 3 has 80-slot rows.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>

#include "device_common.h"
#include "internal.h"
#include "lds_common.h"
#include "tensor_pattern.h"

namespace spingtp {
namespace {

constexpr int kUnrolledWaves = 4;

template <typename P, int I, int NA, int NB, int NO>
__device__ __forceinline__ void entry_step(const float (&a)[NA], const float (&b)[NB], float (&o)[2][NO], float& p,
                                           const float* __restrict__ val) {
    constexpr pattern::Entry e = P::list.e[I];
    constexpr bool fresh = I == 0 || P::list.e[I == 0 ? 0 : I - 1].a != e.a || P::list.e[I == 0 ? 0 : I - 1].b != e.b;
    if constexpr (fresh) p = a[e.a] * b[e.b];
    o[e.half][e.o] = fmaf(val[I], p, o[e.half][e.o]);
}

template <typename P, int BASE, int NA, int NB, int NO, int... I>
__device__ __forceinline__ void entry_chunk(const float (&a)[NA], const float (&b)[NB], float (&o)[2][NO], float& p,
                                            const float* __restrict__ val, std::integer_sequence<int, I...>) {
    (entry_step<P, BASE + I>(a, b, o, p, val), ...);
}

// entries BASE .. n - 1, 64 at a time
template <typename P, int BASE, int NA, int NB, int NO>
__device__ __forceinline__ void entry_chunks(const float (&a)[NA], const float (&b)[NB], float (&o)[2][NO], float& p,
                                             const float* __restrict__ val) {
    if constexpr (BASE < P::list.n) {
        constexpr int N = P::list.n - BASE < 64 ? P::list.n - BASE : 64;
        entry_chunk<P, BASE>(a, b, o, p, val, std::make_integer_sequence<int, N>{});
        entry_chunks<P, BASE + 64>(a, b, o, p, val);
    }
}

// the wave's rows u0 .. u0 + nvalid - 1 through its LDS tile into one register row per lane
template <int N, typename TIO>
__device__ __forceinline__ void unrolled_rows(const TIO* __restrict__ src, int nvalid, float* tile, int lane,
                                              float (&dst)[N]) {
    if (nvalid == 64) load_full_tile<N, N | 1, 64, 64>(src, tile, lane);
    else load_tile<N, N | 1>(src, nvalid, tile, lane, 64);
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < N; ++k) dst[k] = lane < nvalid ? tile[lane * (N | 1) + k] : 0.f;
    wave_lds_order();
}

// dtype (uniform): 0 fp32, 1 bf16 rows (one instantiation for both: the unrolled body is the
// same and large)
template <typename P>
__global__ __launch_bounds__(64 * kUnrolledWaves) void spingtp_fwd_unrolled_kernel(const void* __restrict__ a,
                                                                                   const void* __restrict__ b,
                                                                                   void* __restrict__ out,
                                                                                   int64_t units, int dtype,
                                                                                   const float* __restrict__ val) {
    constexpr int N = P::N;
    __shared__ float lds[kUnrolledWaves][64 * (N | 1)];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t u0 = (static_cast<int64_t>(blockIdx.x) * kUnrolledWaves + wave) * 64;
    if (u0 >= units) return;  // no workgroup barrier below
    const int nvalid = static_cast<int>(units - u0 < 64 ? units - u0 : 64);
    float* tile = lds[wave];
    float ra[N], rb[N], ro[2][N];
    if (dtype == 0) {
        unrolled_rows<N>(static_cast<const float*>(a) + u0 * N, nvalid, tile, lane, ra);
        unrolled_rows<N>(static_cast<const float*>(b) + u0 * N, nvalid, tile, lane, rb);
    } else {
        unrolled_rows<N>(static_cast<const uint16_t*>(a) + u0 * N, nvalid, tile, lane, ra);
        unrolled_rows<N>(static_cast<const uint16_t*>(b) + u0 * N, nvalid, tile, lane, rb);
    }
#pragma unroll
    for (int k = 0; k < N; ++k) ro[0][k] = ro[1][k] = 0.f;
    float p = 0.f;
    entry_chunks<P, 0>(ra, rb, ro, p, val);
#pragma unroll
    for (int k = 0; k < N; ++k) tile[lane * (N | 1) + k] = ro[0][k] + ro[1][k];
    wave_lds_order();
    if (dtype == 0) store_tile<N, N | 1>(static_cast<float*>(out) + u0 * N, nvalid, tile, lane, 64);
    else store_tile<N, N | 1>(static_cast<uint16_t*>(out) + u0 * N, nvalid, tile, lane, 64);
}

template <typename P>
hipError_t launch_unrolled(const void* a, const void* b, void* out, int64_t units, int dtype, const float* val,
                           hipStream_t stream) {
    const int64_t blocks = (units + 64 * kUnrolledWaves - 1) / (64 * kUnrolledWaves);
    if (blocks > 0x7fffffff || val == nullptr || dtype < 0 || dtype > 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(spingtp_fwd_unrolled_kernel<P>, dim3(static_cast<unsigned>(blocks)), dim3(64 * kUnrolledWaves),
                       0, stream, a, b, out, units, dtype, val);
    return hipGetLastError();
}

template <int L, int BASIS>
constexpr UnrolledKernel unrolled_kernel() {
    using P0 = pattern::Pattern<L, 2, BASIS, 0>;
    using P1 = pattern::Pattern<L, 2, BASIS, 1>;
    return UnrolledKernel{{P0::list.n, P1::list.n, P1::list.n},
                          {P0::list.e, P1::list.e, P1::list.e},
                          {&launch_unrolled<P0>, &launch_unrolled<P1>, &launch_unrolled<P1>}};
}

template <int BASIS>
const UnrolledKernel* find_unrolled(int L) {
    static const UnrolledKernel k[2] = {unrolled_kernel<1, BASIS>(), unrolled_kernel<2, BASIS>()};
    return L >= 1 && L <= 2 ? &k[L - 1] : nullptr;
}

}  // namespace
}  // namespace spingtp
