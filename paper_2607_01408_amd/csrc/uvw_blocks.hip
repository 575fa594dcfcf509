// Fully connected SpinGTP product (mode uvw of App. E.1; Sec. 3.5 eq. spin_gtp) and its
// gradients for irrep blocks up to kUvwzMaxD slots wide (degree <= 3), on the matrix cores
// with fp32 operands and sums.  Wider blocks run on the kernels of forward_uvw.hip.
//
// Per edge n and second-input channel v the tensor is contracted with x2 once,
//   K_p[k1, k3] = sum_k2 T[k1, k2, k3] x2[n, v, k2]        (path p = (rho1, rho2 -> rho3)),
// and everything else is dense products on the raw input blocks:
//   out[n, w, k3]    = sum_p sum_k1 K_p[k1, k3] sum_u W[p, u, v, w] x1[n, u, k1],
//   grad_x1[n, u, k1] = sum_p sum_k3 K_p[k1, k3] sum_w W[p, u, v, w] g[n, w, k3],
//   grad_x2[n, v, k2] = sum_p sum_(k1, k3) T[k1, k2, k3] sum_u x1[n, u, k1] sum_w W[p, u, v, w] g[n, w, k3],
//   grad_W[p, u, v, w] = sum_n sum_k3 (sum_k1 x1[n, u, k1] K_p[k1, k3]) g[n, w, k3].
// The inner channel sums are v_mfma_f32_16x16x4f32 / 32x32x2f32 products whose operands are
// the weights (registers, straight from memory) and input blocks staged in LDS once per
// block, not once per path; the contraction with K or T runs on the vector ALU on the
// accumulators.  No per-path operand goes through LDS and no barrier is met per path, which
// is what set the pace of the kernels with per-path operands (forward_uvw.hip).  Measured at
// (2, 2, 2), 1,024 edges, U = W = 64, V = 1, paper basis (123 paths), against those:
//   forward and grad_x1 92 us each (404), grad_x2 122 (633), grad_W 150 (814);
// the matrix products alone take 26 us each at the fp32 matrix rate.  What is left is vector
// work (staging and the contraction, ten instructions per matrix instruction) in the first
// three and the reads of the row blocks in grad_W.  Non-finite inputs: K is dense over a path's
// (k1, k3), so a NaN that comes out may be one of its zeros times an Inf or NaN; such results
// are formed again from the tensor's entries (mix_entries), so an Inf or NaN reaches the slots
// that it has an entry with and no others.
//
// Table (build_uvw_blocks_table): see internal.h.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_common.h"
#include "internal.h"
#include "lds_common.h"

namespace spingtp {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kZE = 16;    // edges of a tile: the N dimension of the 16x16x4 products
constexpr int kZS = 17;    // LDS stride of one (channel, slot) row of kZE edges
constexpr int kZA = 64;    // input channels staged at once, in two halves (one per K split)
constexpr int kZP = 4;     // paths whose K is in LDS at once
constexpr int kZThreads = 512;

__device__ __forceinline__ uint32_t lo16(uint32_t w) { return w & 0xffffu; }
__device__ __forceinline__ uint32_t hi16(uint32_t w) { return w >> 16; }

// floats between the k_out rows of K at one edge (16-byte reads where more than one slot)
constexpr __host__ __device__ int k_stride(int d) { return d == 1 ? 1 : (d == 3 ? 4 : 8); }

// rows [n0, n0 + edges) of x2 channel v into XB[e][stx], with a zero column at ncb (the
// padding entries of the records point there) and zero rows past N
__device__ __forceinline__ void stage_x2(const float* __restrict__ xb, int64_t n0, int64_t N, int V, int v, int ncb,
                                         int stx, int edges, float* XB, int tid, int nthr) {
    for (int i = tid; i < edges * stx; i += nthr) {
        const int e = i / stx, k = i - e * stx;
        const int64_t n = n0 + e;
        XB[i] = (k < ncb && n < N) ? xb[(n * V + v) * ncb + k] : 0.f;
    }
}

// channels a0 .. a0 + kZA - 1, slots [o, o + D) of the tile's rows into X[(a D + k) kZS + e],
// 32 threads per edge; every load of a thread is issued before its first LDS write
template <int D>
__device__ __forceinline__ void stage_block(const float* __restrict__ x, int64_t n0, int64_t N, int A, int nc, int a0,
                                            int o, float* X, int tid) {
    constexpr int IT = kZA * D / 32;
    const int e = tid >> 5, rem = tid & 31;
    const float* __restrict__ row = x + ((n0 + e) * A + a0) * nc + o;
    float v[IT];
    int a = rem / D, k = rem - a * D;
    const int live = n0 + e < N ? A - a0 : 0;  // channels of this edge
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        v[t] = a < live ? row[a * nc + k] : 0.f;
        a += 32 / D;
        k += 32 % D;
        if (k >= D) {
            k -= D;
            ++a;
        }
    }
    float* dst = X + rem * kZS + e;
#pragma unroll
    for (int t = 0; t < IT; ++t) dst[32 * kZS * t] = v[t];
}

// K[k1, k3] of one entry record (two x2 slots and values) at one edge's x2 row
__device__ __forceinline__ float contract_record(const v4u& r, const float* xrow) {
    return fmaf(__uint_as_float(r[3]), xrow[r[2]], __uint_as_float(r[1]) * xrow[r[0]]);
}

// The channel of K step s of lane quarter q within a 32-channel half: steps 4 S .. 4 S + 3
// of a lane are four consecutive channels, so weights contiguous in it load 16 bytes at once.
__device__ __forceinline__ int k_channel(int s, int q) { return 16 * (s >> 2) + 4 * q + (s & 3); }

struct MixArgs {
    const float *xa, *xb, *wt;
    float* out;
    int64_t N, sv, ps;
    uint32_t sa, so;           // weight of (p, a, v, o) at p ps + a sa + v sv + o so
    int A, V, O, nca, ncb, nco;
    int dmax;                  // widest block of either side
    bool vec;                  // sa = 1 and four consecutive weights are 16-byte aligned
    const uint32_t* tab;
    int role;                  // 0: forward (a = x1 blocks), 1: grad_x1 (a = grad_out blocks)
};

// Forward and grad_x1.  A workgroup owns 16 edges, one output block and 16 NWG output
// channels; wave (wg, ks) owns channels 16 wg .. + 15 and half ks of every 64 staged input
// channels (the halves are added in LDS at the end, in a fixed order).  Per (output block,
// input block) pair the input block and the K of its paths are staged; then per path a wave
// runs d_in x 8 products of 16 channels x 16 edges x 4 and adds K times the result to its
// output accumulators.  16-edge tiles, because at 1,024 edges 32-edge tiles leave most SIMDs
// without a wave; two K halves, because the blocks differ in paths by 10x and halving the
// longest chain is worth the second reduction.
struct MixWave {
    int e, q, ks, o_lane, v, stx;
    int64_t n0;
    float *X, *Kt, *XB;
    bool on, o_full;  // some, all of the wave's output channels exist
};

// stage_block for a width known at run time (uniform)
__device__ __forceinline__ void stage_width(int d, const float* __restrict__ x, int64_t n0, int64_t N, int A, int nc,
                                            int a0, int o, float* X, int tid) {
    switch (d) {
        case 1: stage_block<1>(x, n0, N, A, nc, a0, o, X, tid); break;
        case 3: stage_block<3>(x, n0, N, A, nc, a0, o, X, tid); break;
        case 5: stage_block<5>(x, n0, N, A, nc, a0, o, X, tid); break;
        default: stage_block<7>(x, n0, N, A, nc, a0, o, X, tid); break;
    }
}

// The eight K-step weights of a lane's row: channels a .. a + 3 and a + 16 .. a + 19 of
// `count`, at off + channel * sa past the uniform base (32-bit offsets: the launch checks
// the range).  full (uniform): every lane's row and channels exist; vec: sa = 1 and the
// groups of four are 16-byte aligned; nks: K steps in use.
__device__ __forceinline__ void load_weights(const float* __restrict__ base, uint32_t off, uint32_t sa, int a,
                                             int count, bool row_ok, bool full, bool vec, int nks, float (&w)[8]) {
#pragma unroll
    for (int S4 = 0; S4 < 2; ++S4) {
        if (vec) {
            v4f t = {0.f, 0.f, 0.f, 0.f};
            if (full || (row_ok && a + 16 * S4 < count)) t = *reinterpret_cast<const v4f*>(base + (off + a + 16 * S4));
#pragma unroll
            for (int i = 0; i < 4; ++i) w[4 * S4 + i] = t[i];
        } else if (full) {
#pragma unroll
            for (int i = 0; i < 4; ++i) w[4 * S4 + i] = base[off + (a + 16 * S4 + i) * sa];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w[4 * S4 + i] = (row_ok && (S4 == 0 || nks > 4) && a + 16 * S4 + i < count)
                                    ? base[off + (a + 16 * S4 + i) * sa]
                                    : 0.f;
        }
    }
}

// One (output block, input block) pair: stage, then its paths.
template <int DO>
__device__ __forceinline__ void mix_stage(const MixArgs& P, const MixWave& M, int wtid, const uint32_t* __restrict__ S,
                                          const v4u* __restrict__ refs, v4f (&out)[DO]) {
    constexpr int KD = k_stride(DO);
    const int o_in = static_cast<int>(lo16(S[0])), d_in = static_cast<int>(hi16(S[0])), np = static_cast<int>(S[2]);
    const v4u* __restrict__ ref = refs + S[1];
    const bool o_ok = M.o_lane < P.O;
    // S[3] is 0, which the compiler does not know: adding multiples of it to an index keeps
    // the staging addresses from being computed ahead of the loops and held in registers
    // (hundreds of spills otherwise)
    const int zero = static_cast<int>(S[3]);
    for (int p0 = 0; p0 < np; p0 += kZP) {
        const int pn = np - p0 < kZP ? np - p0 : kZP;
        for (int a0 = 0; a0 < P.A; a0 += kZA) {
            const int tid = wtid + zero * (p0 + a0);
            __syncthreads();  // the previous group's reads are done (and XB is written)
            if (p0 == 0 || P.A > kZA)
                stage_width(d_in, P.xa, M.n0, P.N, P.A, P.nca, a0, o_in, M.X, tid);
            if (a0 == 0) {
                for (int i = tid >> 4; i < d_in * DO; i += kZThreads / 16) {
                    const int ki = i / DO, ko = i - ki * DO, e = tid & 15;
                    v4u r[kZP];
#pragma unroll
                    for (int j = 0; j < kZP; ++j)
                        if (j < pn)
                            r[j] = *reinterpret_cast<const v4u*>(P.tab + ref[p0 + j][1] +
                                                                 4 * (P.role == 0 ? i : ko * d_in + ki));
#pragma unroll
                    for (int j = 0; j < kZP; ++j)
                        if (j < pn)
                            M.Kt[((j * d_in + ki) * kZE + e) * KD + ko] = contract_record(r[j], M.XB + e * M.stx);
                }
            }
            __syncthreads();
            const int left = P.A - a0 - 32 * M.ks;
            const int nks = left <= 0 || !M.on ? 0 : (left <= 16 ? 4 : 8);
            if (nks == 0) continue;
            const int a_lane = a0 + 32 * M.ks + 4 * M.q;
            const bool full = left >= 32 && M.o_full;
            auto load = [&](int j, float (&w)[8]) {
                load_weights(P.wt + static_cast<int64_t>(ref[p0 + j][0]) * P.ps + M.v * P.sv,
                             static_cast<uint32_t>(M.o_lane) * P.so, P.sa, a_lane, P.A, o_ok, full, P.vec, nks, w);
            };
            float w[8], wn[8];
            load(0, w);
            const int as = d_in * kZS;  // between the rows of adjacent channels
#pragma unroll 1
            for (int j = 0; j < pn; ++j) {
                if (j + 1 < pn) load(j + 1, wn);
                const float* xk = M.X + (32 * M.ks + 4 * M.q) * as + M.e;
                const float* kr = M.Kt + (j * d_in * kZE + M.e) * KD;
#pragma unroll 1
                for (int ki = 0; ki < d_in; ++ki) {
                    float b[8], kv[DO];
#pragma unroll
                    for (int s = 0; s < 8; ++s)
                        if (s < 4 || nks > 4) b[s] = xk[(16 * (s >> 2) + (s & 3)) * as];
#pragma unroll
                    for (int k = 0; k < DO; ++k) kv[k] = kr[k];
                    v4f z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < 4; ++s) z = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], b[s], z, 0, 0, 0);
                    if (nks > 4) {
#pragma unroll
                        for (int s = 4; s < 8; ++s) z = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], b[s], z, 0, 0, 0);
                    }
#pragma unroll
                    for (int k = 0; k < DO; ++k)
#pragma unroll
                        for (int c = 0; c < 4; ++c) out[k][c] = fmaf(kv[k], z[c], out[k][c]);
                    xk += kZS;
                    kr += kZE * KD;
                }
#pragma unroll
                for (int s = 0; s < 8; ++s) w[s] = wn[s];
            }
        }
    }
}

// A NaN from the dense products, again from the tensor's entries alone: an Inf or NaN meets
// the zeros of K between slots that no entry couples, and 0 Inf is NaN.  Sums of values that are
// finite or truly coupled never take this path (a spurious term is always a NaN), and once the
// sum is a NaN it stays one.
__device__ __forceinline__ float mix_entries(const MixArgs& P, const uint32_t* __restrict__ blk, int64_t n, int o,
                                             int ko) {
    const uint32_t* __restrict__ tab = P.tab;
    const int d_out = static_cast<int>(hi16(blk[0]));
    float s = 0.f;
    for (int v = 0; v < P.V; ++v)
        for (uint32_t st = blk[1]; st < blk[1] + blk[2]; ++st) {
            const uint32_t* __restrict__ S = tab + tab[5 + 4 * P.role] + 4 * st;
            const int o_in = static_cast<int>(lo16(S[0])), d_in = static_cast<int>(hi16(S[0]));
            for (uint32_t j = S[1]; j < S[1] + S[2]; ++j) {
                const uint32_t* __restrict__ ref = tab + tab[6 + 4 * P.role] + 4 * j;
                for (int ki = 0; ki < d_in; ++ki) {
                    const uint32_t* __restrict__ r = tab + ref[1] + 4 * (P.role == 0 ? ki * d_out + ko : ko * d_in + ki);
                    for (int t = 0; t < 2; ++t) {
                        const float val = __uint_as_float(r[2 * t + 1]);
                        if (val == 0.f) continue;
                        const float b = val * P.xb[(n * P.V + v) * P.ncb + r[2 * t]];
                        const float* __restrict__ w = P.wt + ref[0] * P.ps + v * P.sv + static_cast<int64_t>(o) * P.so;
                        for (int a = 0; a < P.A && s == s; ++a)
                            s = fmaf(w[static_cast<int64_t>(a) * P.sa], P.xa[(n * P.A + a) * P.nca + o_in + ki] * b, s);
                    }
                }
            }
        }
    return s;
}

template <int DO>
__device__ __forceinline__ void mix_block(const MixArgs& P, const uint32_t* __restrict__ blk, float* sm) {
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int nthr = kZThreads, nwg = 4;  // nwg: waves per K half
    const int wg = wave % nwg, ks = wave / nwg;
    const int e = lane & 15, q = lane >> 4;
    const int64_t n0 = static_cast<int64_t>(blockIdx.x) * kZE;
    const int o0 = static_cast<int>(blockIdx.z) * 16 * nwg;
    const int stx = (P.ncb + 1) | 1;
    float* X = sm;
    float* Kt = X + kZA * P.dmax * kZS;
    float* XB = Kt + kZP * P.dmax * kZE * k_stride(P.dmax);
    const uint32_t* __restrict__ tab = P.tab;
    const uint32_t* __restrict__ stages = tab + tab[5 + 4 * P.role];
    const v4u* __restrict__ refs = reinterpret_cast<const v4u*>(tab + tab[6 + 4 * P.role]);
    const int st0 = static_cast<int>(blk[1]), nst = static_cast<int>(blk[2]);
    const int o_out = static_cast<int>(lo16(blk[0]));
    // o_lane: the row this lane's weights belong to
    MixWave M{e, q, ks, o0 + 16 * wg + e, 0, stx, n0, X, Kt, XB, o0 + 16 * wg < P.O, o0 + 16 * wg + 16 <= P.O};

    v4f out[DO];
#pragma unroll
    for (int k = 0; k < DO; ++k) out[k] = v4f{0.f, 0.f, 0.f, 0.f};

    if (nst > 0)
        for (int v = 0; v < P.V; ++v) {
            M.v = v;
            __syncthreads();
            stage_x2(P.xb, n0, P.N, P.V, v, P.ncb, stx, kZE, XB, tid, nthr);
            for (int st = st0; st < st0 + nst; ++st) {
                const uint32_t* __restrict__ S = stages + 4 * st;
                mix_stage<DO>(P, M, tid, S, refs, out);
            }
        }

    // the second K half's sums, then the first's added, through an [edge][channel][slot] tile
    // in LDS, so that the rows leave in runs of consecutive addresses
    const int no = 16 * nwg;
    const int ste = no * DO + 1;
    __syncthreads();
    float* t = X + e * ste + (16 * wg + 4 * q) * DO;
    if (ks == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < DO; ++k) t[r * DO + k] = out[k][r];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < DO; ++k) t[r * DO + k] += out[k][r];
    }
    __syncthreads();
    const int on = P.O - o0 < no ? P.O - o0 : no;
    const int per = on * DO;
    bool again = false;
    for (int i = tid; i < kZE * per; i += nthr) {
        const int er = i / per, rem = i - er * per;
        const int o = rem / DO, k = rem - o * DO;
        const int64_t n = n0 + er;
        const float v = X[er * ste + rem];
        if (n < P.N) P.out[(n * P.O + o0 + o) * P.nco + o_out + k] = v;
        again |= v != v;
    }
    if (again)
        for (int i = tid; i < kZE * per; i += nthr) {
            const int er = i / per, rem = i - er * per;
            const int o = rem / DO, k = rem - o * DO;
            const int64_t n = n0 + er;
            const float v = X[er * ste + rem];
            if (n < P.N && v != v) P.out[(n * P.O + o0 + o) * P.nco + o_out + k] = mix_entries(P, blk, n, o0 + o, k);
        }
}

// DM: the widest output block
template <int DM>
__global__ __launch_bounds__(kZThreads, DM <= 5 ? 4 : 2) void spingtp_uvwz_mix_kernel(MixArgs P) {
    extern __shared__ float sm[];
    const uint32_t* blk = P.tab + P.tab[3 + 4 * P.role] + 4 * blockIdx.y;
    switch (hi16(blk[0])) {  // uniform over the workgroup
        case 1: mix_block<1>(P, blk, sm); break;
        case 3: mix_block<3>(P, blk, sm); break;
        case 5: mix_block<5>(P, blk, sm); break;
        default:
            if constexpr (DM > 5) mix_block<7>(P, blk, sm);
            break;
    }
}

struct GradX2Args {
    const float *x1, *g, *wt;
    float* gx2;
    int64_t N;
    int U, V, W, nc1, nc2, nco, d1max, wch;  // wch: channels w of grad_out staged at once (16 or 32)
    bool vec;
    const uint32_t* tab;
};

// One path of grad_x2 for a wave's 16 u rows and 16 edges: Q[k3] = sum_w W g (matrix
// cores), then acc[k2] += T[k1, k3, k2] x1[u, k1] Q[u, k3] over the lane's four rows.
template <int D2, int D3>
__device__ __forceinline__ void grad_x2_path(const float (&w)[8], int nks, const float* G, int nco, int o3,
                                             const float* X, int d1, const float* __restrict__ T, int e, int q, int ug,
                                             float (&acc)[D2]) {
    v4f z[D3];
#pragma unroll
    for (int k = 0; k < D3; ++k) z[k] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 8; ++s)
        if (s < 4 || nks > 4) {
            const float* gr = G + (k_channel(s, q) * nco + o3) * kZS + e;
#pragma unroll
            for (int k = 0; k < D3; ++k) z[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], gr[k * kZS], z[k], 0, 0, 0);
        }
    const float* xr = X + (16 * ug + 4 * q) * d1 * kZS + e;
    for (int k1 = 0; k1 < d1; ++k1) {
        float xv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) xv[r] = xr[(r * d1 + k1) * kZS];
#pragma unroll
        for (int k = 0; k < D3; ++k) {
            const float pr = fmaf(xv[3], z[k][3], fmaf(xv[2], z[k][2], fmaf(xv[1], z[k][1], xv[0] * z[k][0])));
#pragma unroll
            for (int k2 = 0; k2 < D2; ++k2) acc[k2] = fmaf(T[(k1 * D3 + k) * D2 + k2], pr, acc[k2]);
        }
    }
}

// grad_x2[n, v, k2 of the block] from the tensor's entries (see mix_entries)
__device__ __forceinline__ float grad_x2_entries(const GradX2Args& P, const uint32_t* __restrict__ blk, int64_t n, int v,
                                                 int k2) {
    const uint32_t* __restrict__ tab = P.tab;
    const int d2 = static_cast<int>(hi16(blk[0]));
    float s = 0.f;
    for (uint32_t st = blk[1]; st < blk[1] + blk[2]; ++st) {
        const uint32_t* __restrict__ S = tab + tab[5 + 8] + 4 * st;
        const int o1 = static_cast<int>(lo16(S[0])), d1 = static_cast<int>(hi16(S[0]));
        for (uint32_t j = S[1]; j < S[1] + S[2]; ++j) {
            const uint32_t* __restrict__ ref = tab + tab[6 + 8] + 4 * j;
            const int o3 = static_cast<int>(lo16(ref[3])), d3 = static_cast<int>(hi16(ref[3]));
            for (int i = 0; i < d1 * d3; ++i) {
                const float val = __uint_as_float(tab[ref[2] + i * d2 + k2]);
                if (val == 0.f) continue;
                for (int u = 0; u < P.U && s == s; ++u) {
                    const float a = val * P.x1[(n * P.U + u) * P.nc1 + o1 + i / d3];
                    const float* __restrict__ w =
                        P.wt + ((static_cast<int64_t>(ref[0]) * P.U + u) * P.V + v) * static_cast<int64_t>(P.W);
                    for (int c = 0; c < P.W; ++c) s = fmaf(w[c], a * P.g[(n * P.W + c) * P.nco + o3 + i % d3], s);
                }
            }
        }
    }
    return s;
}

// grad_x2.  A workgroup owns 16 edges, one block of x2 and one channel v; wave (ug, ph)
// takes the u rows 16 ug .. + 15 of every 64 and every second path (ph).  grad_out rows of
// wch channels are staged whole (every path reads some block of them), the x1 block once
// per rho1.  The lane sums meet at the end: two shuffles over the row quarters, then the
// eight waves' sums added in wave order.
template <int D2, int DM>
__device__ __forceinline__ void grad_x2_block(const GradX2Args& P, const uint32_t* __restrict__ blk, float* sm) {
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ug = wave & 3, ph = wave >> 2;
    const int e = lane & 15, q = lane >> 4;
    const int64_t n0 = static_cast<int64_t>(blockIdx.x) * kZE;
    const int v = static_cast<int>(blockIdx.z);
    float* G = sm;
    float* X = G + P.wch * P.nco * kZS;
    const uint32_t* __restrict__ tab = P.tab;
    const uint32_t* __restrict__ stages = tab + tab[5 + 8];
    const v4u* __restrict__ refs = reinterpret_cast<const v4u*>(tab + tab[6 + 8]);
    const int st0 = static_cast<int>(blk[1]), nst = static_cast<int>(blk[2]);
    const int o2 = static_cast<int>(lo16(blk[0]));
    const int64_t VW = static_cast<int64_t>(P.V) * P.W, UVW = P.U * VW;

    float acc[D2];
#pragma unroll
    for (int k = 0; k < D2; ++k) acc[k] = 0.f;

    if (nst > 0)
        for (int w0 = 0; w0 < P.W; w0 += P.wch) {
            __syncthreads();
            {  // whole rows of wch channels: G[(w nco + k) kZS + e], eight loads in flight
                const int per = P.wch * P.nco;
                const int live = (P.W - w0 < P.wch ? P.W - w0 : P.wch) * P.nco;
                for (int e8 = 0; e8 < kZE; e8 += 8)
                    for (int i = tid; i < per; i += kZThreads) {
                        float t[8];
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const int64_t n = n0 + e8 + r;
                            t[r] = (n < P.N && i < live) ? P.g[(n * P.W + w0) * P.nco + i] : 0.f;
                        }
#pragma unroll
                        for (int r = 0; r < 8; ++r) G[i * kZS + e8 + r] = t[r];
                    }
            }
            const int left = P.W - w0 < P.wch ? P.W - w0 : P.wch;
            const int nks = left <= 16 ? 4 : 8;
            for (int u0 = 0; u0 < P.U; u0 += kZA) {
                int turn = 0;  // alternates the half that takes the first path of a stage
                const int u_lane = u0 + 16 * ug + e;
                for (int st = st0; st < st0 + nst; ++st) {
                    const uint32_t* __restrict__ S = stages + 4 * st;
                    const int o1 = static_cast<int>(lo16(S[0])), d1 = static_cast<int>(hi16(S[0]));
                    const int np = static_cast<int>(S[2]);
                    const v4u* __restrict__ ref = refs + S[1];
                    const int st_tid = tid + static_cast<int>(S[3]);  // S[3] is 0 (see mix_stage)
                    __syncthreads();
                    stage_width(d1, P.x1, n0, P.N, P.U, P.nc1, u0, o1, X, st_tid);
                    __syncthreads();
                    const bool full = left == 32 && u0 + 16 * ug + 16 <= P.U;
                    auto load = [&](int j, float (&w)[8]) {
                        load_weights(P.wt + static_cast<int64_t>(ref[j][0]) * UVW + static_cast<int64_t>(v) * P.W,
                                     static_cast<uint32_t>(u_lane) * static_cast<uint32_t>(VW), 1u, w0 + 4 * q,
                                     nks > 4 ? P.W : (P.W < w0 + 16 ? P.W : w0 + 16), u_lane < P.U, full, P.vec, nks,
                                     w);
                    };
                    float w[8], wn[8];
                    int j = (ph + turn) & 1;
                    if (j < np) load(j, w);
                    for (; j < np; j += 2) {
                        if (j + 2 < np) load(j + 2, wn);
                        const int o3 = static_cast<int>(lo16(ref[j][3]));
                        const float* __restrict__ T = reinterpret_cast<const float*>(tab + ref[j][2]);
                        switch (hi16(ref[j][3])) {
                            case 1: grad_x2_path<D2, 1>(w, nks, G, P.nco, o3, X, d1, T, e, q, ug, acc); break;
                            case 3: grad_x2_path<D2, 3>(w, nks, G, P.nco, o3, X, d1, T, e, q, ug, acc); break;
                            case 5: grad_x2_path<D2, 5>(w, nks, G, P.nco, o3, X, d1, T, e, q, ug, acc); break;
                            default:
                                if constexpr (DM > 5)
                                    grad_x2_path<D2, 7>(w, nks, G, P.nco, o3, X, d1, T, e, q, ug, acc);
                                break;
                        }
#pragma unroll
                        for (int s = 0; s < 8; ++s) w[s] = wn[s];
                    }
                    turn += np & 1;
                }
            }
        }

#pragma unroll
    for (int k = 0; k < D2; ++k) {
        acc[k] += __shfl_xor(acc[k], 16);
        acc[k] += __shfl_xor(acc[k], 32);
    }
    __syncthreads();
    if (q == 0) {
#pragma unroll
        for (int k = 0; k < D2; ++k) sm[(wave * kZE + e) * D2 + k] = acc[k];
    }
    __syncthreads();
    for (int i = tid; i < kZE * D2; i += kZThreads) {
        const int er = i / D2, k = i - er * D2;
        float s = 0.f;
        for (int w = 0; w < 8; ++w) s += sm[(w * kZE + er) * D2 + k];
        if (n0 + er >= P.N) continue;
        if (s != s) s = grad_x2_entries(P, blk, n0 + er, v, k);
        P.gx2[((n0 + er) * P.V + v) * P.nc2 + o2 + k] = s;
    }
}

// DM: the widest block of x2 and of the output
template <int DM>
__global__ __launch_bounds__(kZThreads, DM <= 5 ? 4 : 2) void spingtp_uvwz_grad_x2_kernel(GradX2Args P) {
    extern __shared__ float sm[];
    const uint32_t* blk = P.tab + P.tab[3 + 8] + 4 * blockIdx.y;
    switch (hi16(blk[0])) {
        case 1: grad_x2_block<1, DM>(P, blk, sm); break;
        case 3: grad_x2_block<3, DM>(P, blk, sm); break;
        case 5: grad_x2_block<5, DM>(P, blk, sm); break;
        default:
            if constexpr (DM > 5) grad_x2_block<7, DM>(P, blk, sm);
            break;
    }
}

struct GradWArgs {
    const float *x1, *x2, *g;
    float* gw;
    int64_t N;
    int U, V, W, nc1, nc2, nco, d1max, d3max;
    unsigned tiles;  // 32 x 32 tiles of (u, w); workgroup = unit x tile
    const uint32_t* tab;
};

constexpr int kGE = 8;          // edges of a wave's turn in the weight gradient
constexpr int kGWaves = 16;
constexpr int kGThreads = 64 * kGWaves;

// D consecutive floats of a row (4-byte aligned: one or two wide loads)
template <int D>
__device__ __forceinline__ void load_row(const float* __restrict__ p, float (&v)[D]) {
    __builtin_memcpy(v, p, sizeof(v));
}

// grad_W[path][u][v][w] from the tensor's entries (see mix_entries)
__device__ __forceinline__ float grad_w_entries(const GradWArgs& P, const uint32_t* __restrict__ unit,
                                                const uint32_t* __restrict__ rec, int u, int v, int w) {
    const int o1 = static_cast<int>(lo16(unit[0])), d1 = static_cast<int>(hi16(unit[0]));
    const int o3 = static_cast<int>(lo16(unit[1])), d3 = static_cast<int>(hi16(unit[1]));
    float s = 0.f;
    for (int64_t n = 0; n < P.N && s == s; ++n)
        for (int i = 0; i < d1 * d3; ++i)
            for (int t = 0; t < 2; ++t) {
                const float val = __uint_as_float(rec[4 * i + 2 * t + 1]);
                if (val == 0.f) continue;
                s = fmaf(val * P.x1[(n * P.U + u) * P.nc1 + o1 + i / d3] * P.x2[(n * P.V + v) * P.nc2 + rec[4 * i + 2 * t]],
                         P.g[(n * P.W + w) * P.nco + o3 + i % d3], s);
            }
    return s;
}

// grad_W.  A workgroup owns up to kUvwzUnitPaths paths of one (rho1, rho3) pair, 32 channels
// u, 32 channels w and one v; wave i takes the edges 8 (i + 16 t) .. + 7 of turn t, and
// nothing is shared between the waves until their sums are added, in wave order, at the end
// (so no barrier in the loop).  A lane holds channel u = w = lane % 32 of one edge of a pair:
// the operand R[u] = sum_k1 x1[u, k1] K[k1, k3] of the product is formed in registers from
// the lane's own x1 block, the other operand is its grad_out block, two edges per K step;
// K comes from LDS, formed by the wave for its 8 edges.  Paths of a pair share the row
// loads: each block is a few slots of a 100-byte row, so row loads (a line each) are the
// next bound after the products.
template <int D1, int D3>
__device__ __forceinline__ void grad_w_unit(const GradWArgs& P, const uint32_t* __restrict__ unit, float* sm) {
    constexpr int KD = k_stride(D1), PER = D1 * D3;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, half = lane >> 5;
    const uint32_t* __restrict__ tab = P.tab;
    const v4u* __restrict__ ref = reinterpret_cast<const v4u*>(tab + tab[17]) + unit[2];
    const int np = static_cast<int>(unit[3]);
    const int tile = static_cast<int>(blockIdx.x % P.tiles);
    const int o1 = static_cast<int>(lo16(unit[0])), o3 = static_cast<int>(lo16(unit[1]));
    const int v = static_cast<int>(blockIdx.y);
    const int wt = (P.W + 31) / 32;
    const int u0 = tile / wt * 32, w0 = tile % wt * 32;
    const int stx = (P.nc2 + 1) | 1;
    v4u* R = reinterpret_cast<v4u*>(sm);                      // the paths' records
    float* Kt = sm + 4 * kUvwzUnitPaths * P.d1max * P.d3max +  // this wave's [path][k3][edge][KD]
                wave * kUvwzUnitPaths * P.d3max * kGE * k_stride(P.d1max);
    float* XB = sm + 4 * kUvwzUnitPaths * P.d1max * P.d3max +  // this wave's x2 rows
                kGWaves * kUvwzUnitPaths * P.d3max * kGE * k_stride(P.d1max) + wave * kGE * stx;

    for (int i = tid; i < np * PER; i += kGThreads)
        R[i] = *reinterpret_cast<const v4u*>(tab + ref[i / PER][1] + 4 * (i % PER));
    v16f acc[kUvwzUnitPaths];
#pragma unroll
    for (int j = 0; j < kUvwzUnitPaths; ++j) acc[j] = v16f{};
    __syncthreads();

    // lanes past U or W repeat the last channel's rows (their sums are not stored)
    const int64_t ur = u0 + c < P.U ? u0 + c : P.U - 1, wr = w0 + c < P.W ? w0 + c : P.W - 1;
    const float* __restrict__ xp = P.x1 + ur * P.nc1 + o1;
    const float* __restrict__ gp = P.g + wr * P.nco + o3;
    const int64_t xs = static_cast<int64_t>(P.U) * P.nc1, gs = static_cast<int64_t>(P.W) * P.nco;
    float xv[2][D1], gv[2][D3];
    auto fetch = [&](int64_t n, float (&x)[D1], float (&g)[D3]) {
        if (n < P.N) {
            load_row<D1>(xp + n * xs, x);
            load_row<D3>(gp + n * gs, g);
        } else {
#pragma unroll
            for (int k = 0; k < D1; ++k) x[k] = 0.f;
#pragma unroll
            for (int k = 0; k < D3; ++k) g[k] = 0.f;
        }
    };
    const int64_t n_first = kGE * wave;
    fetch(n_first + half, xv[0], gv[0]);
    for (int64_t n0 = n_first; n0 < P.N; n0 += kGE * kGWaves) {
        // this turn's K, in the wave's own LDS region: the last turn's reads of K and x2 are
        // ordered before these writes, the x2 rows before the lanes that form K, K before its use
        wave_lds_order();
        for (int i = lane; i < kGE * stx; i += 64) {
            const int e = i / stx, k = i - e * stx;
            XB[i] = (k < P.nc2 && n0 + e < P.N) ? P.x2[((n0 + e) * P.V + v) * P.nc2 + k] : 0.f;
        }
        wave_lds_order();
        for (int i = lane >> 3; i < np * PER; i += 8) {
            const int j = i / PER, rem = i - j * PER, k1 = rem / D3, k3 = rem - k1 * D3;
            const int e = lane & 7;
            Kt[((j * D3 + k3) * kGE + e) * KD + k1] = contract_record(R[i], XB + e * stx);
        }
        wave_lds_order();
#pragma unroll
        for (int s = 0; s < kGE / 2; ++s) {
            const int e = 2 * s + half;
            const int64_t next = s + 1 < kGE / 2 ? n0 + e + 2 : n0 + kGE * kGWaves + half;
            fetch(next, xv[(s + 1) & 1], gv[(s + 1) & 1]);
#pragma unroll
            for (int k3 = 0; k3 < D3; ++k3) {
#pragma unroll
                for (int j = 0; j < kUvwzUnitPaths; ++j)
                    if (j < np) {
                        const float* kr = Kt + ((j * D3 + k3) * kGE + e) * KD;
                        float r = xv[s & 1][0] * kr[0];
#pragma unroll
                        for (int k = 1; k < D1; ++k) r = fmaf(xv[s & 1][k], kr[k], r);
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(r, gv[s & 1][k3], acc[j], 0, 0, 0);
                    }
            }
        }
    }

    // accumulator element i of lane l: u = u0 + 8 (i / 4) + 4 (l / 32) + i % 4, w = w0 + l % 32;
    // the other waves' sums through LDS (16 x 64 floats each), added by wave 0 in wave order
    const int64_t VW = static_cast<int64_t>(P.V) * P.W;
    float* red = sm;
    bool again = false;
#pragma unroll
    for (int j = 0; j < kUvwzUnitPaths; ++j) {
        if (j >= np) break;
        __syncthreads();
        if (wave > 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) red[((wave - 1) * 16 + i) * 64 + lane] = acc[j][i];
        }
        __syncthreads();
        if (wave == 0 && w0 + c < P.W) {
            float* __restrict__ dst = P.gw + static_cast<int64_t>(ref[j][0]) * P.U * VW +
                                      static_cast<int64_t>(v) * P.W + w0 + c;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float s = acc[j][i];
                for (int w = 0; w < kGWaves - 1; ++w) s += red[(w * 16 + i) * 64 + lane];
                const int u = u0 + 8 * (i >> 2) + 4 * half + (i & 3);
                if (u < P.U) {
                    dst[u * VW] = s;
                    again |= s != s;
                }
            }
        }
    }
    if (again)
#pragma unroll 1
        for (int i = 0; i < 16 * np; ++i) {
            const uint32_t* __restrict__ path = tab + tab[17] + 4 * (unit[2] + i / 16);
            const int u = u0 + 8 * (i % 16 >> 2) + 4 * half + (i & 3);
            if (u >= P.U) continue;
            float* dst = P.gw + (static_cast<int64_t>(path[0]) * P.U + u) * VW + static_cast<int64_t>(v) * P.W + w0 + c;
            if (*dst != *dst) *dst = grad_w_entries(P, unit, tab + path[1], u, v, w0 + c);
        }
}

__global__ __launch_bounds__(kGThreads, 4) void spingtp_uvwz_grad_w_kernel(GradWArgs P) {
    extern __shared__ float sm[];
    const uint32_t* unit = P.tab + P.tab[15] + 4 * (blockIdx.x / P.tiles);
    switch (hi16(unit[0]) << 4 | hi16(unit[1])) {
#define SPINGTP_UNIT(a, b) \
    case (a << 4 | b): grad_w_unit<a, b>(P, unit, sm); break;
#define SPINGTP_UNITS(a) SPINGTP_UNIT(a, 1) SPINGTP_UNIT(a, 3) SPINGTP_UNIT(a, 5) SPINGTP_UNIT(a, 7)
        SPINGTP_UNITS(1) SPINGTP_UNITS(3) SPINGTP_UNITS(5) SPINGTP_UNITS(7)
#undef SPINGTP_UNITS
#undef SPINGTP_UNIT
        default: break;  // no other width is tabulated
    }
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

size_t mix_lds(const UvwzShape& s, int ncb) {
    return sizeof(float) * (kZA * s.dmax * kZS + kZP * s.dmax * kZE * k_stride(s.dmax) + kZE * ((ncb + 1) | 1));
}

size_t grad_w_lds(const UvwzShape& s) {
    const size_t words = 4 * kUvwzUnitPaths * s.d1max * s.d3max +
                         kGWaves * kGE * (kUvwzUnitPaths * s.d3max * k_stride(s.d1max) + ((s.nc2 + 1) | 1));
    const size_t red = (kGWaves - 1) * 16 * 64;
    return sizeof(float) * (words > red ? words : red);
}

// channels of grad_out the x2 gradient stages at once (0: its tiles do not fit)
int grad_x2_wch(const UvwzShape& s) {
    for (int wch : {32, 16})
        if (sizeof(float) * kZS * (wch * s.nco + kZA * s.d1max) <= (wch > 16 ? 80 : 160) * 1024) return wch;
    return 0;
}

template <int DM>
hipError_t launch_mix(const MixArgs& P, dim3 grid, size_t lds, hipStream_t stream) {
    if (lds > 65536) {
        const hipError_t e = raise_lds_limit<&spingtp_uvwz_mix_kernel<DM>>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(spingtp_uvwz_mix_kernel<DM>, grid, dim3(kZThreads), lds, stream, P);
    return hipGetLastError();
}

template <int DM>
hipError_t launch_grad_x2(const GradX2Args& P, dim3 grid, size_t lds, hipStream_t stream) {
    if (lds > 65536) {
        const hipError_t e = raise_lds_limit<&spingtp_uvwz_grad_x2_kernel<DM>>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(spingtp_uvwz_grad_x2_kernel<DM>, grid, dim3(kZThreads), lds, stream, P);
    return hipGetLastError();
}

}  // namespace

bool uvwz_fits(const UvwzShape& s) {
    return s.dmax >= 1 && s.dmax <= kUvwzMaxD && mix_lds(s, s.nc2) <= 160 * 1024 && grad_w_lds(s) <= 160 * 1024 &&
           grad_x2_wch(s) > 0;
}

hipError_t launch_uvwz_mix(const float* xa, const float* xb, const float* w, float* out, int64_t N, int A, int V, int O,
                           int64_t sa, int64_t sv, int64_t so, int64_t ps, const UvwzShape& s, const uint32_t* table,
                           int role, hipStream_t stream) {
    const int64_t gx = (N + kZE - 1) / kZE;
    const int blocks = s.blocks[role];
    if (gx == 0 || O == 0 || blocks == 0) return hipSuccess;
    const int64_t gz = (O + 63) / 64;
    if (gx > 0x7fffffff || blocks > 65535 || gz > 65535) return hipErrorInvalidValue;
    const bool vec = sa == 1 && ps % 4 == 0 && sv % 4 == 0 && so % 4 == 0 && A % 4 == 0 && aligned16(w);
    // (an empty input side is not read: no channel v is visited)
    MixArgs P{xa, xb, w, out, N, sv, ps, static_cast<uint32_t>(sa), static_cast<uint32_t>(so), A, A > 0 ? V : 0, O, role == 0 ? s.nc1 : s.nco, s.nc2, role == 0 ? s.nco : s.nc1,
              s.dmax, vec, table, role};
    const size_t lds = mix_lds(s, s.nc2);
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(blocks), static_cast<unsigned>(gz));
    return (role == 0 ? s.d3max : s.d1max) <= 5 ? launch_mix<5>(P, grid, lds, stream)
                                                : launch_mix<7>(P, grid, lds, stream);
}

hipError_t launch_uvwz_grad_x2(const float* x1, const float* g, const float* w, float* gx2, int64_t N, int U, int V,
                               int W, const UvwzShape& s, const uint32_t* table, hipStream_t stream) {
    const int64_t gx = (N + kZE - 1) / kZE;
    if (gx == 0 || V == 0 || s.blocks[2] == 0) return hipSuccess;
    if (gx > 0x7fffffff || s.blocks[2] > 65535 || V > 65535) return hipErrorInvalidValue;
    const int wch = grad_x2_wch(s);
    GradX2Args P{x1, g, w, gx2, N, U, V, U > 0 ? W : 0, s.nc1, s.nc2, s.nco, s.d1max, wch, W % 4 == 0 && aligned16(w), table};
    const size_t lds = sizeof(float) * kZS * (wch * s.nco + kZA * s.d1max);
    if (wch == 0) return hipErrorInvalidValue;
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(s.blocks[2]), static_cast<unsigned>(V));
    return s.d2max <= 5 && s.d3max <= 5 ? launch_grad_x2<5>(P, grid, lds, stream)
                                        : launch_grad_x2<7>(P, grid, lds, stream);
}

hipError_t launch_uvwz_grad_w(const float* x1, const float* x2, const float* g, float* gw, int64_t N, int U, int V,
                              int W, const UvwzShape& s, const uint32_t* table, hipStream_t stream) {
    if (s.units == 0 || U == 0 || V == 0 || W == 0) return hipSuccess;
    const int64_t tiles = static_cast<int64_t>((U + 31) / 32) * ((W + 31) / 32);
    if (tiles * s.units > 0x7fffffff || V > 65535) return hipErrorInvalidValue;
    GradWArgs P{x1,    x2,    g,     gw,      N,       U,       V, W, s.nc1,
                s.nc2, s.nco, s.d1max, s.d3max, static_cast<unsigned>(tiles), table};
    const size_t lds = grad_w_lds(s);
    if (lds > 65536) {
        const hipError_t e = raise_lds_limit<&spingtp_uvwz_grad_w_kernel>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(spingtp_uvwz_grad_w_kernel,
                       dim3(static_cast<unsigned>(tiles * s.units), static_cast<unsigned>(V)), dim3(kGThreads), lds, stream, P);
    return hipGetLastError();
}

}  // namespace spingtp
