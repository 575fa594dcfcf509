// Per-channel path-weighted product with the edge input shared by the channels (App. E.1, mode
// uvu; spingtp_forward_v1_weighted, spingtp_forward_depthwise and their gradients), for irrep
// blocks up to kCwMaxD slots wide (degree <= 3).  Other shapes, and x2 per unit, run on the
// entry-list kernels of backward_v1w.hip.
//
// x2 is the same for every channel of an edge, so the tensor is contracted with it once per
// edge, K_p[k1, k3] = sum_k2 T x2[n, k2] (path p = (rho1, rho2 -> rho3)), and each channel then
// works on K, dense in a path's (k1, k3):
//   out[c, k3] = sum_p W[c, p] sum_k1 x1[c, k1] K_p[k1, k3],
//   t_p[c, k1] = sum_k3 K_p[k1, k3] g[c, k3],  gx1[c, k1] = sum_p W[c, p] t_p[c, k1],
//   gW[c, p]  += sum_k1 x1[c, k1] t_p[c, k1],
//   gx2[k2]    = sum_p sum_(k1, k3) T M_p[k1, k3],  M_p[k1, k3] = sum_c W[c, p] x1[c, k1] g[c, k3],
// the channel sums M on the matrix cores (fp32 operands and sums).  Per path and channel that
// is one weight, d1 (or d3) row values and d1 d3 / 4 broadcast reads of K, where the entry-list
// kernels gather three values from LDS per tensor entry.
// Mapping: a workgroup owns a 64-channel tile (one channel per lane) and a range of edges, its
// waves split the output blocks (schedule in the table, balanced by cost).  K of a block is
// formed by its wave in a wave-private LDS region, so the only barriers are those around an
// edge's rows, and the next edge's rows are in flight meanwhile.  Measured, 1,024 edges, us,
// against the entry lists: (2, 2, 2), 64 channels, paper basis: forward 50 -> 23, gradients
// 157 -> 59 (the kernel alone); (1, 3, 3), 128 channels, parity basis: forward 55 -> 38, gradients
// 184 -> 60.  One edge alone takes 11 us (25) and 22 us (73).  What bounds it now: the gradients'
// weight and sum tiles leave room for one workgroup per CU in the paper basis, and its waves
// stand at a wait or barrier for 55 to 61 % of their cycles (the vector ALU issues on 32 to 39 %;
// 2 to 5 % wait for the LDS pipe to take an instruction).  Non-finite inputs: K is dense over a path's (k1, k3), so a NaN that comes
// out may be one of its zeros times an Inf or NaN; such results are formed again from the
// tensor's entries (cw_entries), so an Inf or NaN reaches the slots that it has an entry with
// and no others.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_common.h"
#include "internal.h"
#include "lds_common.h"

namespace spingtp {
namespace {

constexpr int kCwLanes = 64;

__device__ __forceinline__ int cw_stride(int n) { return (n + 1) | 1; }  // odd, with a zero column
int cw_stride_host(int n) { return (n + 1) | 1; }

__device__ __forceinline__ float cw_load(const float* p) { return *p; }
__device__ __forceinline__ float cw_load(const uint16_t* p) { return bf16_to_f32(*p); }
__device__ __forceinline__ void cw_store(float* p, float v) { *p = v; }
__device__ __forceinline__ void cw_store(uint16_t* p, float v) { *p = f32_to_bf16(v); }

// floats between the rows of K at one contracted slot
constexpr __host__ __device__ int cw_k_stride(int d) { return d == 1 ? 1 : (d == 3 ? 4 : 8); }

// rows [0, nrows) of a contiguous [nrows][nc] block into LDS rows of stride st, eight loads in
// flight per thread; (r, c) advance by THR elements without a division per element
template <int THR, typename TIO>
__device__ __forceinline__ void cw_stage(const TIO* __restrict__ src, int nrows, int nc, int st, float* dst, int tid) {
    const int n = nrows * nc;
    int r = tid / nc, c = tid - r * nc;
    const int dr = THR / nc, dc = THR - dr * nc;
    for (int e0 = tid; e0 < n; e0 += 8 * THR) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = e0 + i * THR < n ? cw_load(src + e0 + i * THR) : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (e0 + i * THR < n) dst[r * st + c] = v[i];
            r += dr;
            c += dc;
            if (c >= nc) {
                c -= nc;
                ++r;
            }
        }
    }
}

// The same in two steps, so that an edge's rows are in flight while the previous edge is worked
// on: the first 8 THR elements of the block wait in registers, the rest (long rows) are read
// when they are put away.
template <int THR, typename TIO>
struct CwRows {
    float v[8];
    __device__ __forceinline__ void fetch(const TIO* __restrict__ src, int n, int tid) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i * THR < n) v[i] = tid + i * THR < n ? cw_load(src + tid + i * THR) : 0.f;
    }
    __device__ __forceinline__ void put(const TIO* __restrict__ src, int n, int nc, int st, float* dst, int tid) const {
        int r = tid / nc, c = tid - r * nc;
        const int dr = THR / nc, dc = THR - dr * nc;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i * THR >= n) break;
            if (tid + i * THR < n) dst[r * st + c] = v[i];
            r += dr;
            c += dc;
            if (c >= nc) {
                c -= nc;
                ++r;
            }
        }
        for (int e = tid + 8 * THR; e < n; e += THR) dst[(e / nc) * st + e % nc] = cw_load(src + e);
    }
};

// sum over the tensor's entries of output slot k of W[p] value in[slot] x2[slot], from the blocks
// (output blocks of the forward, x1 blocks of the gradients) whose references, items follow
// at words 1 and 2 of `at`; nv second inputs x2v apart with weights wslice apart.  For results
// that came out NaN (a spurious term is always a NaN; once the sum is one it stays so).
// From global memory: other waves may be filling the LDS tiles with the next edge.
template <typename TIO>
__device__ __forceinline__ float cw_entries(const uint32_t* __restrict__ tab, const uint32_t* __restrict__ at, int n_blocks,
                                            int k, const float* __restrict__ w, const TIO* __restrict__ in,
                                            const TIO* __restrict__ x2, int nv, int64_t x2v, int64_t wslice) {
    float s = 0.f;
    for (int b = 0; b < n_blocks; ++b) {
        const uint32_t* __restrict__ blk = tab + at[0] + 8 * b;
        const int o = k - static_cast<int>(blk[0] & 0xffffu), d_o = static_cast<int>(blk[0] >> 16);
        if (o < 0 || o >= d_o) continue;
        const uint32_t* __restrict__ item = tab + at[2] + 4 * blk[3] + 4 * o;
        uint32_t left = blk[5];  // references of width 1, 3, 5, 7 still to come, a byte each
        int d_i = 1;
        for (uint32_t j = blk[1]; j < blk[1] + blk[2]; ++j) {
            while ((left & 0xffu) == 0) {
                left >>= 8;
                d_i += 2;
            }
            --left;
            const uint32_t* __restrict__ ref = tab + at[1] + 4 * j;
            for (int i = 0; i < d_i; ++i, item += 4 * d_o)
                for (int t = 0; t < 2 && s == s; ++t) {
                    const float val = __uint_as_float(item[1 + t]);
                    if (val == 0.f) continue;
                    const uint32_t k2 = t == 0 ? item[0] & 0xffffu : item[0] >> 16;
                    const float a = val * cw_load(in + ref[1] + i);
                    for (int v = 0; v < nv; ++v)
                        s = fmaf(w[v * wslice + ref[0]], a * cw_load(x2 + v * x2v + k2), s);
                }
        }
    }
    return s;
}

// grad_W[channel c][path p] over the edges [n0, n1), likewise
template <typename TIO>
__device__ __forceinline__ float cw_weight_entries(const uint32_t* __restrict__ tab, int n_blocks, int p, int64_t n0,
                                                   int64_t n1, int64_t C, int64_t c, const TIO* __restrict__ x1, int nc1,
                                                   const TIO* __restrict__ g, int nco, const TIO* __restrict__ x2,
                                                   int64_t x2s) {
    float s = 0.f;
    for (int b = 0; b < n_blocks; ++b) {
        const uint32_t* __restrict__ blk = tab + tab[13] + 8 * b;
        const int o = static_cast<int>(blk[0] & 0xffffu), d_o = static_cast<int>(blk[0] >> 16);
        const uint32_t* __restrict__ item = tab + tab[15] + 4 * blk[3];
        uint32_t left = blk[5];
        int d_i = 1;
        for (uint32_t j = blk[1]; j < blk[1] + blk[2]; ++j) {
            while ((left & 0xffu) == 0) {
                left >>= 8;
                d_i += 2;
            }
            --left;
            const uint32_t* __restrict__ ref = tab + tab[14] + 4 * j;
            if (ref[0] == static_cast<uint32_t>(p))
                for (int64_t n = n0; n < n1 && s == s; ++n)
                    for (int i = 0; i < 2 * d_i * d_o; ++i) {
                        const uint32_t* __restrict__ it = item + 4 * (i >> 1);
                        const float val = __uint_as_float(it[1 + (i & 1)]);
                        if (val == 0.f) continue;
                        const uint32_t k2 = (i & 1) == 0 ? it[0] & 0xffffu : it[0] >> 16;
                        s = fmaf(val * cw_load(x1 + (n * C + c) * nc1 + o + (i >> 1) % d_o),
                                 cw_load(x2 + n * x2s + k2) * cw_load(g + (n * C + c) * nco + ref[1] + (i >> 1) / d_o), s);
                    }
            item += 4 * d_i * d_o;
        }
    }
    return s;
}

// entries(r, c): the element from the tensor's entries, for those that are NaN here
template <int THR, typename TIO, typename Entries>
__device__ __forceinline__ void cw_unstage(TIO* __restrict__ dst, int nrows, int nc, int st, const float* src, int second,
                                           int tid, bool add, const Entries& entries) {
    const int n = nrows * nc;
    int r = tid / nc, c = tid - r * nc;
    const int dr = THR / nc, dc = THR - dr * nc;
    for (int e = tid; e < n; e += THR) {
        float v = src[r * st + c];
        if (second) v += src[second + r * st + c];  // the blocks' second parts
        if (__builtin_expect(v != v, 0)) v = entries(r, c);
        cw_store(dst + e, add ? cw_load(dst + e) + v : v);
        r += dr;
        c += dc;
        if (c >= nc) {
            c -= nc;
            ++r;
        }
    }
}

// K of one block: items of {x2 slots, two values, destination}, 64 at a time
__device__ __forceinline__ void cw_form_k(const v4u* __restrict__ items, int n, const float* x2, float* Kt, int lane) {
    for (int i0 = lane; i0 < n; i0 += 256) {
        v4u it[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i0 + 64 * j < n) it[j] = items[i0 + 64 * j];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i0 + 64 * j < n)
                Kt[it[j][3]] = fmaf(__uint_as_float(it[j][2]), x2[it[j][0] >> 16],
                                    __uint_as_float(it[j][1]) * x2[it[j][0] & 0xffffu]);
    }
}

// one row of K (16-byte aligned where it has more than one slot)
template <int D>
__device__ __forceinline__ void cw_k_row(const float* K, float (&k)[D]) {
    if constexpr (D == 1) {
        k[0] = K[0];
    } else {
        float t[cw_k_stride(D)];
#pragma unroll
        for (int i = 0; i < cw_k_stride(D); i += 4) {
            const v4f v = *reinterpret_cast<const v4f*>(K + i);
#pragma unroll
            for (int j = 0; j < 4; ++j) t[i + j] = v[j];
        }
#pragma unroll
        for (int i = 0; i < D; ++i) k[i] = t[i];
    }
}

// The references of a block, one per lane (at most 64), read by readlane: loading each as the
// loop reaches it would cost a memory latency per path.
struct CwRefs {
    uint32_t p, in, k;
};
__device__ __forceinline__ CwRefs cw_load_refs(const v4u* __restrict__ ref, int n, int lane) {
    const v4u r = ref[lane < n ? lane : 0];
    return CwRefs{r[0], r[1], r[2]};
}
__device__ __forceinline__ uint32_t cw_lane(uint32_t v, int j) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), j));
}

// out[k] += w sum_i x[i] K[i][k], the row values already read
template <int DO, int DI>
struct CwPathRows {
    float w, x[DI], k[DI][DO];
    __device__ __forceinline__ void read(const CwRefs& R, int j, const float* W, const float* X, const float* Kt) {
        constexpr int KD = cw_k_stride(DO);
        w = W[cw_lane(R.p, j)];
        const float* xr = X + cw_lane(R.in, j);
        const float* kr = Kt + cw_lane(R.k, j);
#pragma unroll
        for (int i = 0; i < DI; ++i) {
            x[i] = xr[i];
            cw_k_row<DO>(kr + i * KD, k[i]);
        }
    }
    // (the path's own sum first: one chain over all paths and slots rounds more than the entry
    // lists' two)
    __device__ __forceinline__ void add(float (&out)[DO]) const {
#pragma unroll
        for (int c = 0; c < DO; ++c) {
            float y = x[0] * k[0][c];
#pragma unroll
            for (int i = 1; i < DI; ++i) y = fmaf(x[i], k[i][c], y);
            out[c] = fmaf(w, y, out[c]);
        }
    }
};

// references j0 .. j1 - 1, all with DI contracted slots, two at a time (the second one's reads
// cover the first one's arithmetic)
template <int DO, int DI>
__device__ __forceinline__ void cw_fwd_group(const CwRefs& R, int j0, int j1, const float* W, const float* X,
                                             const float* Kt, float (&out)[DO]) {
    int j = j0;
    if constexpr (DO * DI <= 25) {  // (larger pairs would cost a workgroup of occupancy)
#pragma unroll 1
        for (; j + 2 <= j1; j += 2) {
            CwPathRows<DO, DI> a, b;
            a.read(R, j, W, X, Kt);
            b.read(R, j + 1, W, X, Kt);
            a.add(out);
            b.add(out);
        }
    }
#pragma unroll 1
    for (; j < j1; ++j) {
        CwPathRows<DO, DI> a;
        a.read(R, j, W, X, Kt);
        a.add(out);
    }
}

struct CwArgs {
    const void *x1, *x2, *g;
    void *out, *gx1, *gx2;
    const float* wts;
    float *ws_x2, *ws_w;
    int64_t N, C, epg, x2s, x2v, wslice;
    bool add;  // add to out (forward) or gx1 (gradients)
    const uint32_t* tab;
    int kfloats;  // the K region of a wave
};

// One block of the forward: NV second-input channels (K of one at a time), then its row slots.
template <int DO, int NV, int DM>
__device__ __forceinline__ void cw_fwd_block(const uint32_t* __restrict__ blk, const v4u* __restrict__ refs,
                                             const v4u* __restrict__ items, const float* Wr, int wv, const float* X1r,
                                             const float* X2, int st2, float* Kt, float* Or, int lane) {
    float out[DO];
#pragma unroll
    for (int k = 0; k < DO; ++k) out[k] = 0.f;
    const CwRefs R = cw_load_refs(refs + blk[1], static_cast<int>(blk[2]), lane);
    const int e1 = static_cast<int>(blk[5] & 0xffu), e3 = e1 + static_cast<int>((blk[5] >> 8) & 0xffu);
    const int e5 = e3 + static_cast<int>((blk[5] >> 16) & 0xffu), e7 = static_cast<int>(blk[2]);
#pragma unroll 1
    for (int v = 0; v < NV; ++v) {
        const float* Wv = Wr + v * wv;
        wave_lds_order();
        cw_form_k(items + blk[3], static_cast<int>(blk[4]), X2 + v * st2, Kt, lane);
        wave_lds_order();
        cw_fwd_group<DO, 1>(R, 0, e1, Wv, X1r, Kt, out);
        cw_fwd_group<DO, 3>(R, e1, e3, Wv, X1r, Kt, out);
        cw_fwd_group<DO, 5>(R, e3, e5, Wv, X1r, Kt, out);
        if constexpr (DM > 5) cw_fwd_group<DO, 7>(R, e5, e7, Wv, X1r, Kt, out);
    }
    const int o = static_cast<int>(blk[0] & 0xffffu);
#pragma unroll
    for (int k = 0; k < DO; ++k) Or[o + k] = out[k];
}

constexpr int kCwFwdThreads = 64 * kCwFwdWaves;

// DM: the widest block of x1 and of the output
template <typename TIO, int NV, int DM>
__global__ __launch_bounds__(kCwFwdThreads, 4) void spingtp_cw_fwd_kernel(CwArgs P) {
    extern __shared__ float lds[];
    const uint32_t* __restrict__ tab = P.tab;
    const int np = static_cast<int>(tab[0]), nc1 = static_cast<int>(tab[1]), nc2 = static_cast<int>(tab[2]);
    const int nco = static_cast<int>(tab[3]);
    const int stw = cw_stride(np), st1 = cw_stride(nc1), sto = cw_stride(nco), st2 = cw_stride(nc2);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int parts = static_cast<int>(tab[4]);
    float* Kt = lds + wave * P.kfloats;
    float* Wt = lds + kCwFwdWaves * P.kfloats;      // [NV][64][stw]
    float* X1 = Wt + NV * kCwLanes * stw;           // [64][st1]
    float* O = X1 + kCwLanes * st1;                 // [parts][64][sto]
    float* X2 = O + parts * kCwLanes * sto;         // [NV][st2]
    const int64_t c0 = static_cast<int64_t>(blockIdx.y) * kCwLanes;
    const int nch = static_cast<int>(P.C - c0 < kCwLanes ? P.C - c0 : kCwLanes);
    const int64_t n_begin = blockIdx.x * P.epg;
    const int64_t n_end = n_begin + P.epg < P.N ? n_begin + P.epg : P.N;

    // zero columns, rows past nch and slots no path reaches stay zero
    const int total = kCwLanes * (NV * stw + st1 + parts * sto) + NV * st2;
    for (int i = tid; i < total; i += kCwFwdThreads) Wt[i] = 0.f;
    __syncthreads();
    for (int v = 0; v < NV; ++v)
        cw_stage<kCwFwdThreads>(P.wts + v * P.wslice + c0 * np, nch, np, stw, Wt + v * kCwLanes * stw, tid);
    const uint32_t* __restrict__ sched = tab + tab[8];
    const uint32_t* __restrict__ blocks = tab + tab[9];
    const v4u* __restrict__ refs = reinterpret_cast<const v4u*>(tab + tab[10]);
    const v4u* __restrict__ items = reinterpret_cast<const v4u*>(tab + tab[11]);
    const int b0 = static_cast<int>(sched[wave]), b1 = static_cast<int>(sched[wave + 1]);
    const TIO* __restrict__ x1 = static_cast<const TIO*>(P.x1);
    const TIO* __restrict__ x2 = static_cast<const TIO*>(P.x2);
    TIO* __restrict__ out = static_cast<TIO*>(P.out);

    CwRows<kCwFwdThreads, TIO> r1;
    if (n_begin < n_end) r1.fetch(x1 + (n_begin * P.C + c0) * nc1, nch * nc1, tid);
    for (int64_t n = n_begin; n < n_end; ++n) {
        const int64_t row0 = n * P.C + c0;
        r1.put(x1 + row0 * nc1, nch * nc1, nc1, st1, X1, tid);
        for (int i = tid; i < NV * nc2; i += kCwFwdThreads) {
            const int v = i / nc2, k = i - v * nc2;
            X2[v * st2 + k] = cw_load(x2 + n * P.x2s + v * P.x2v + k);
        }
        __syncthreads();  // (also: the previous edge's output rows have left)
        if (n + 1 < n_end) r1.fetch(x1 + (row0 + P.C) * nc1, nch * nc1, tid);
        for (int b = b0; b < b1; ++b) {
            const uint32_t* __restrict__ blk = blocks + 8 * b;
            const float *Wr = Wt + lane * stw, *X1r = X1 + lane * st1;
            float* Or = O + (blk[6] * kCwLanes + lane) * sto;
            switch (blk[0] >> 16) {
                case 1: cw_fwd_block<1, NV, DM>(blk, refs, items, Wr, kCwLanes * stw, X1r, X2, st2, Kt, Or, lane); break;
                case 3: cw_fwd_block<3, NV, DM>(blk, refs, items, Wr, kCwLanes * stw, X1r, X2, st2, Kt, Or, lane); break;
                case 5: cw_fwd_block<5, NV, DM>(blk, refs, items, Wr, kCwLanes * stw, X1r, X2, st2, Kt, Or, lane); break;
                default:
                    if constexpr (DM > 5)
                        cw_fwd_block<7, NV, DM>(blk, refs, items, Wr, kCwLanes * stw, X1r, X2, st2, Kt, Or, lane);
                    break;
            }
        }
        __syncthreads();
        cw_unstage<kCwFwdThreads>(out + row0 * nco, nch, nco, sto, O, parts > 1 ? kCwLanes * sto : 0, tid, P.add,
                                  [&](int r, int k) {
                                      return cw_entries(tab, tab + 9, static_cast<int>(sched[kCwFwdWaves]), k,
                                                        P.wts + (c0 + r) * np, x1 + (row0 + r) * nc1, x2 + n * P.x2s,
                                                        NV, P.x2v, P.wslice);
                                  });
    }
}

// t[k1] = sum_k3 K[k3][k1] g[k3]; gx[k1] += w t[k1]; returns sum_k1 x1[k1] t[k1]
template <int D1, int D3>
__device__ __forceinline__ float cw_bwd_path(const CwPathRows<D1, D3>& r, const float (&x)[D1], float (&gx)[D1]) {
    float t[D1];
#pragma unroll
    for (int i = 0; i < D3; ++i)
#pragma unroll
        for (int k = 0; k < D1; ++k) t[k] = i == 0 ? r.x[i] * r.k[i][k] : fmaf(r.x[i], r.k[i][k], t[k]);
    float s = x[0] * t[0];
    gx[0] = fmaf(r.w, t[0], gx[0]);
#pragma unroll
    for (int k = 1; k < D1; ++k) {
        s = fmaf(x[k], t[k], s);
        gx[k] = fmaf(r.w, t[k], gx[k]);
    }
    return s;
}

template <int D1, int D3>
__device__ __forceinline__ void cw_bwd_group(const CwRefs& R, int j0, int j1, const float* W, float* GW, const float* G,
                                             const float* Kt, const float (&x)[D1], float (&gx)[D1]) {
    int j = j0;
    if constexpr (D1 * D3 <= 15) {
#pragma unroll 1
        for (; j + 2 <= j1; j += 2) {  // (the paths of a block are distinct)
            CwPathRows<D1, D3> a, b;
            a.read(R, j, W, G, Kt);
            b.read(R, j + 1, W, G, Kt);
            float *pa = GW + cw_lane(R.p, j), *pb = GW + cw_lane(R.p, j + 1);
            const float ga = *pa, gb = *pb;
            const float sa = cw_bwd_path<D1, D3>(a, x, gx), sb = cw_bwd_path<D1, D3>(b, x, gx);
            *pa = ga + sa;
            *pb = gb + sb;
        }
    }
#pragma unroll 1
    for (; j < j1; ++j) {
        CwPathRows<D1, D3> a;
        a.read(R, j, W, G, Kt);
        float* pa = GW + cw_lane(R.p, j);
        *pa += cw_bwd_path<D1, D3>(a, x, gx);
    }
}

template <int D1, int DM>
__device__ __forceinline__ void cw_bwd_block(const uint32_t* __restrict__ blk, const v4u* __restrict__ refs,
                                             const v4u* __restrict__ items, const float* Wr, float* GWr,
                                             const float* X1r, const float* Gr, const float* X2, float* Kt, float* GXr,
                                             int lane) {
    const CwRefs R = cw_load_refs(refs + blk[1], static_cast<int>(blk[2]), lane);
    const int e1 = static_cast<int>(blk[5] & 0xffu), e3 = e1 + static_cast<int>((blk[5] >> 8) & 0xffu);
    const int e5 = e3 + static_cast<int>((blk[5] >> 16) & 0xffu), e7 = static_cast<int>(blk[2]);
    const int o = static_cast<int>(blk[0] & 0xffffu);
    wave_lds_order();
    cw_form_k(items + blk[3], static_cast<int>(blk[4]), X2, Kt, lane);
    wave_lds_order();
    float x[D1], gx[D1];
#pragma unroll
    for (int k = 0; k < D1; ++k) {
        x[k] = X1r[o + k];
        gx[k] = 0.f;
    }
    cw_bwd_group<D1, 1>(R, 0, e1, Wr, GWr, Gr, Kt, x, gx);
    cw_bwd_group<D1, 3>(R, e1, e3, Wr, GWr, Gr, Kt, x, gx);
    cw_bwd_group<D1, 5>(R, e3, e5, Wr, GWr, Gr, Kt, x, gx);
    if constexpr (DM > 5) cw_bwd_group<D1, 7>(R, e5, e7, Wr, GWr, Gr, Kt, x, gx);
#pragma unroll
    for (int k = 0; k < D1; ++k) GXr[o + k] = gx[k];
}


// M_p[k1, k3] of 16 rows (p, k1) and the 16 columns from slot col0 of the output (columns past
// the spin's slots hold values no entry reads): v_mfma_f32_16x16x4f32 over the 64 channels.
// B (the grad_out columns) is the same for all tiles of a spin.

// DM: the widest block of x1 and of the output; NW: waves (16 where one workgroup's LDS takes
// more than half a CU's, else 8 so that two run: (2, 2, 2) paper basis 8 -> 16 waves 76 -> 59 us,
// (1, 3, 3) parity basis 62 against 74, 1,024 edges)
template <typename TIO, int DM, int NW>
__global__ __launch_bounds__(64 * NW, 4) void spingtp_cw_bwd_kernel(CwArgs P) {
    constexpr int kCwBwdWaves = NW, kCwBwdThreads = 64 * NW;
    extern __shared__ float lds[];
    const uint32_t* __restrict__ tab = P.tab;
    const int np = static_cast<int>(tab[0]), nc1 = static_cast<int>(tab[1]), nc2 = static_cast<int>(tab[2]);
    const int nco = static_cast<int>(tab[3]);
    const int stw = cw_stride(np), st1 = cw_stride(nc1), sto = cw_stride(nco), st2 = cw_stride(nc2);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = static_cast<int>(tab[20]);
    float* Kt = lds + wave * P.kfloats;
    float* M = lds + kCwBwdWaves * P.kfloats;  // [tile][16 rows][16 columns]
    float* Wt = M + ntiles * 256;              // [64][stw]
    float* GW = Wt + kCwLanes * stw;           // [64][stw]
    float* X1 = GW + kCwLanes * stw;           // [64][st1]
    const int parts = static_cast<int>(tab[5]);
    float* GX = X1 + kCwLanes * st1;           // [parts][64][st1]
    float* G = GX + parts * kCwLanes * st1;    // [64][sto]
    float* X2 = G + kCwLanes * sto;            // [st2]
    const int64_t c0 = static_cast<int64_t>(blockIdx.y) * kCwLanes;
    const int nch = static_cast<int>(P.C - c0 < kCwLanes ? P.C - c0 : kCwLanes);
    const int64_t n_begin = blockIdx.x * P.epg;
    const int64_t n_end = n_begin + P.epg < P.N ? n_begin + P.epg : P.N;

    const int total = kCwLanes * (2 * stw + (1 + parts) * st1 + sto) + st2;
    for (int i = tid; i < total; i += kCwBwdThreads) Wt[i] = 0.f;
    __syncthreads();
    cw_stage<kCwBwdThreads>(P.wts + c0 * np, nch, np, stw, Wt, tid);
    const uint32_t* __restrict__ sched = tab + tab[12];
    const uint32_t* __restrict__ blocks = tab + tab[13];
    const v4u* __restrict__ refs = reinterpret_cast<const v4u*>(tab + tab[14]);
    const v4u* __restrict__ items = reinterpret_cast<const v4u*>(tab + tab[15]);
    const uint32_t* __restrict__ rows = tab + tab[16];   // 16 per tile: path | x1 slot << 16
    const uint32_t* __restrict__ cols = tab + tab[17];   // per tile: its first output slot
    const uint32_t* __restrict__ seg = tab + tab[18];    // nc2 + 1: entries of each x2 slot
    const uint32_t* __restrict__ ent = tab + tab[19];    // entries: index into M, value
    const int b0 = static_cast<int>(sched[wave]), b1 = static_cast<int>(sched[wave + 1]);
    const int t0 = static_cast<int>(tab[tab[21] + wave]), t1 = static_cast<int>(tab[tab[21] + wave + 1]);
    const TIO* __restrict__ x1 = static_cast<const TIO*>(P.x1);
    const TIO* __restrict__ x2 = static_cast<const TIO*>(P.x2);
    const TIO* __restrict__ g = static_cast<const TIO*>(P.g);
    TIO* __restrict__ gx1 = static_cast<TIO*>(P.gx1);
    const int cl = lane & 15, q = lane >> 4;

    CwRows<kCwBwdThreads, TIO> r1, rg;
    if (n_begin < n_end) {
        r1.fetch(x1 + (n_begin * P.C + c0) * nc1, nch * nc1, tid);
        rg.fetch(g + (n_begin * P.C + c0) * nco, nch * nco, tid);
    }
    for (int64_t n = n_begin; n < n_end; ++n) {
        const int64_t row0 = n * P.C + c0;
        r1.put(x1 + row0 * nc1, nch * nc1, nc1, st1, X1, tid);
        rg.put(g + row0 * nco, nch * nco, nco, sto, G, tid);
        for (int k = tid; k < nc2; k += kCwBwdThreads) X2[k] = cw_load(x2 + n * P.x2s + k);
        __syncthreads();
        if (n + 1 < n_end) {
            r1.fetch(x1 + (row0 + P.C) * nc1, nch * nc1, tid);
            rg.fetch(g + (row0 + P.C) * nco, nch * nco, tid);
        }
        for (int b = b0; b < b1; ++b) {
            const uint32_t* __restrict__ blk = blocks + 8 * b;
            const float *Wr = Wt + lane * stw, *X1r = X1 + lane * st1, *Gr = G + lane * sto;
            float *GWr = GW + lane * stw, *GXr = GX + (blk[6] * kCwLanes + lane) * st1;
            switch (blk[0] >> 16) {
                case 1: cw_bwd_block<1, DM>(blk, refs, items, Wr, GWr, X1r, Gr, X2, Kt, GXr, lane); break;
                case 3: cw_bwd_block<3, DM>(blk, refs, items, Wr, GWr, X1r, Gr, X2, Kt, GXr, lane); break;
                case 5: cw_bwd_block<5, DM>(blk, refs, items, Wr, GWr, X1r, Gr, X2, Kt, GXr, lane); break;
                default:
                    if constexpr (DM > 5) cw_bwd_block<7, DM>(blk, refs, items, Wr, GWr, X1r, Gr, X2, Kt, GXr, lane);
                    break;
            }
        }
        // the channel sums M of this wave's tiles (the waves with few paths have more of them)
        for (int t = t0; t < t1; ++t) {
            const int col = static_cast<int>(cols[t]) + cl;
            const float* gc = G + q * sto + (col < nco ? col : nco);  // (the zero column past the rows)
            const uint32_t rw = rows[16 * t + cl];
            const float* wr = Wt + q * stw + (rw & 0xffffu);
            const float* xr = X1 + q * st1 + (rw >> 16);
            // eight chains of 8 channels (four at a time) and their tree: one or two long chains
            // round more than the entry lists' tree over the lanes
            v4f sum[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4f acc[4];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int s = 8 * h + i;
                    const v4f c = i < 4 ? v4f{0.f, 0.f, 0.f, 0.f} : acc[i & 3];
                    acc[i & 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[4 * s * stw] * xr[4 * s * st1], gc[4 * s * sto],
                                                                      c, 0, 0, 0);
                }
                sum[h] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) M[t * 256 + (4 * q + r) * 16 + cl] = sum[0][r] + sum[1][r];
        }
        __syncthreads();
        // gx2: 16 lanes per x2 slot take its entries in turn; their sums are added by shuffles
        // in a fixed order
        for (int k0 = 0; k0 < nc2; k0 += kCwBwdThreads / 16) {
            const int k = k0 + (tid >> 4);
            float s = 0.f;
            if (k < nc2)
                for (uint32_t e = seg[k] + cl; e < seg[k + 1]; e += 16)
                    s = fmaf(__uint_as_float(ent[2 * e + 1]), M[ent[2 * e]], s);
#pragma unroll
            for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off, 16);
            if (cl == 0 && k < nc2) {
                if (gridDim.y == 1) cw_store(static_cast<TIO*>(P.gx2) + n * P.x2s + k, s);
                else P.ws_x2[(blockIdx.y * P.N + n) * nc2 + k] = s;
            }
        }
        cw_unstage<kCwBwdThreads>(gx1 + row0 * nc1, nch, nc1, st1, GX, parts > 1 ? kCwLanes * st1 : 0, tid, P.add,
                                  [&](int r, int k) {
                                      return cw_entries(tab, tab + 13, static_cast<int>(sched[kCwBwdWaves]), k,
                                                        P.wts + (c0 + r) * np, g + (row0 + r) * nco, x2 + n * P.x2s, 1,
                                                        0, 0);
                                  });
        // (the next edge's rows go into X1, G and X2, which no wave reads past the barrier above;
        // its M and GX writes come after the next barrier)
    }
    __syncthreads();
    if (n_end > n_begin)
        for (int i = tid; i < np * kCwLanes; i += kCwBwdThreads) {
            const int p = i >> 6, r = i & 63;
            if (r >= nch) continue;
            float s = GW[r * stw + p];
            if (s != s)  // (see cw_entries)
                s = cw_weight_entries(tab, static_cast<int>(sched[kCwBwdWaves]), p, n_begin, n_end, P.C, c0 + r, x1, nc1,
                                      g, nco, x2, P.x2s);
            P.ws_w[(blockIdx.x * static_cast<int64_t>(np) + p) * P.C + c0 + r] = s;
        }
}

template <typename TIO, int NV, int DM>
hipError_t cw_fwd(const CwArgs& P, dim3 grid, size_t bytes, hipStream_t stream) {
    if (bytes > 65536) {
        const hipError_t e = raise_lds_limit<&spingtp_cw_fwd_kernel<TIO, NV, DM>>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((spingtp_cw_fwd_kernel<TIO, NV, DM>), grid, dim3(kCwFwdThreads), bytes, stream, P);
    return hipGetLastError();
}

template <typename TIO, int DM>
hipError_t cw_fwd_nv(int nv, const CwArgs& P, dim3 grid, size_t bytes, hipStream_t stream) {
    switch (nv) {
        case 1: return cw_fwd<TIO, 1, DM>(P, grid, bytes, stream);
        case 2: return cw_fwd<TIO, 2, DM>(P, grid, bytes, stream);
        case 3: return cw_fwd<TIO, 3, DM>(P, grid, bytes, stream);
        case 4: return cw_fwd<TIO, 4, DM>(P, grid, bytes, stream);
        default: return hipErrorInvalidValue;
    }
}

template <typename TIO, int DM, int NW>
hipError_t cw_bwd(const CwArgs& P, dim3 grid, size_t bytes, hipStream_t stream) {
    if (bytes > 65536) {
        const hipError_t e = raise_lds_limit<&spingtp_cw_bwd_kernel<TIO, DM, NW>>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((spingtp_cw_bwd_kernel<TIO, DM, NW>), grid, dim3(64 * NW), bytes, stream, P);
    return hipGetLastError();
}

template <typename TIO, int DM>
hipError_t cw_bwd_waves(int waves, const CwArgs& P, dim3 grid, size_t bytes, hipStream_t stream) {
    if (waves == 16) return cw_bwd<TIO, DM, 16>(P, grid, bytes, stream);
    return waves == 8 ? cw_bwd<TIO, DM, 8>(P, grid, bytes, stream) : hipErrorInvalidValue;
}

}  // namespace

int cw_fwd_lds_floats(const CwShape& s, int nv) {
    return kCwFwdWaves * s.kfloats[0] +
           kCwLanes * (nv * cw_stride_host(s.np) + cw_stride_host(s.nc1) + s.parts[0] * cw_stride_host(s.nco)) +
           nv * cw_stride_host(s.nc2);
}

int cw_bwd_lds_floats(const CwShape& s) {
    return s.bwd_waves * s.kfloats[1] + s.tiles * 256 +
           kCwLanes * (2 * cw_stride_host(s.np) + (1 + s.parts[1]) * cw_stride_host(s.nc1) + cw_stride_host(s.nco)) +
           cw_stride_host(s.nc2);
}

hipError_t launch_cw_fwd(int dtype, const void* x1, const void* x2, const float* w, void* out, int64_t N, int64_t C,
                         const CwShape& s, const uint32_t* tab, hipStream_t stream, int64_t x2s, bool add, int nv,
                         int64_t x2v, int64_t wslice) {
    const int lds = cw_fwd_lds_floats(s, nv);
    if (lds > kBw1wMaxLdsFloats || tab == nullptr) return hipErrorInvalidValue;
    const int64_t tiles = (C + kCwLanes - 1) / kCwLanes;
    int64_t groups = 0, epg = 0;
    const int per_cu = kBw1wMaxLdsFloats / lds;
    bw1w_groups(N, C, &groups, &epg, 256 * (per_cu > 4 ? 4 : per_cu));
    if (groups == 0 || tiles == 0) return hipSuccess;
    if (groups > 0x7fffffff || tiles > 0xffff) return hipErrorInvalidValue;
    CwArgs P{};
    P.x1 = x1;
    P.x2 = x2;
    P.out = out;
    P.wts = w;
    P.N = N;
    P.C = C;
    P.epg = epg;
    P.x2s = x2s > 0 ? x2s : s.nc2;
    P.x2v = x2v;
    P.wslice = wslice;
    P.add = add;
    P.tab = tab;
    P.kfloats = s.kfloats[0];
    const dim3 grid(static_cast<unsigned>(groups), static_cast<unsigned>(tiles));
    const size_t bytes = static_cast<size_t>(lds) * sizeof(float);
    if (s.dmax <= 5)
        return dtype == 0 ? cw_fwd_nv<float, 5>(nv, P, grid, bytes, stream)
                          : cw_fwd_nv<uint16_t, 5>(nv, P, grid, bytes, stream);
    return dtype == 0 ? cw_fwd_nv<float, 7>(nv, P, grid, bytes, stream)
                      : cw_fwd_nv<uint16_t, 7>(nv, P, grid, bytes, stream);
}

hipError_t launch_cw_bwd(int dtype, const void* x1, const void* x2, const float* w, const void* g, void* gx1, void* gx2,
                         float* ws_x2, float* ws_w, int64_t N, int64_t C, int64_t groups, int64_t epg, const CwShape& s,
                         const uint32_t* tab, hipStream_t stream, int64_t x2s, bool add) {
    const int lds = cw_bwd_lds_floats(s);
    const int64_t tiles = (C + kCwLanes - 1) / kCwLanes;
    if (lds > kBw1wMaxLdsFloats || tab == nullptr || groups > 0x7fffffff || tiles > 0xffff) return hipErrorInvalidValue;
    CwArgs P{};
    P.x1 = x1;
    P.x2 = x2;
    P.g = g;
    P.gx1 = gx1;
    P.gx2 = gx2;
    P.wts = w;
    P.ws_x2 = ws_x2;
    P.ws_w = ws_w;
    P.N = N;
    P.C = C;
    P.epg = epg;
    P.x2s = x2s > 0 ? x2s : s.nc2;
    P.add = add;
    P.tab = tab;
    P.kfloats = s.kfloats[1];
    const dim3 grid(static_cast<unsigned>(groups), static_cast<unsigned>(tiles));
    const size_t bytes = static_cast<size_t>(lds) * sizeof(float);
    if (s.dmax <= 5)
        return dtype == 0 ? cw_bwd_waves<float, 5>(s.bwd_waves, P, grid, bytes, stream)
                          : cw_bwd_waves<uint16_t, 5>(s.bwd_waves, P, grid, bytes, stream);
    return dtype == 0 ? cw_bwd_waves<float, 7>(s.bwd_waves, P, grid, bytes, stream)
                      : cw_bwd_waves<uint16_t, 7>(s.bwd_waves, P, grid, bytes, stream);
}

}  // namespace spingtp
