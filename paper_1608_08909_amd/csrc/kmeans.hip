// k-means sp pivot refinement (paper Section 4.1, "k-means sp"): Lloyd
// iterations over the nodes' hop-distance vectors to the max/min pivots.
//
// Node i's feature vector is y_i = (dist[0][i], ..., dist[k-1][i]).  Cluster
// t is held as the exact integer sum S_t of its members' vectors (in double:
// every sum stays below 2^53) and its size N_t; it starts as y_{p_t}.  One
// pass: every node joins the cluster with the smallest
//     f_t(i) = a_t - (2 B_ti) / N_t,   B_ti = y_i . S_t (an exact integer),
//     a_t = sum_j (S_tj / N_t)^2 in ascending j, no fused multiply-add,
// lowest t on ties; every non-empty cluster's sums are then recomputed (an
// empty one keeps its centroid).  Passes stop when no node moves or after
// max_iters.  New pivot t is the free node with the smallest
// N_t ||y_i||^2 - 2 B_ti (exact 64-bit integers), lowest id on ties, ranks in
// ascending order.
//
// Layout: the sums are feature-major, ST[j * k + t] = S_tj, so that the C
// sums one block needs for feature j are consecutive and wave-uniform: the
// contraction B = Y S^T (2 n k^2 flops per pass) runs as FP64 FMAs whose
// cluster operand comes from scalar loads, one node per lane, C clusters
// per block.  Every product and partial sum is an integer below 2^53, so the
// FMAs are exact in any order.  The assignment itself runs on the 8-bit matrix
// instructions from kKmMatrixMinK pivots on, wherever the distances and sums
// split into few digits (k_km_assign_mx); the passes follow one another on the device, a flag ending
// them, and the host looks at it every kKmBatch passes.
#include <stdlib.h>

#include <climits>
#include <vector>

#include "ssm_internal.h"
#include "wave.h"

namespace ssm {

constexpr int kKmBlock = 256;
constexpr int kKmChunk = 32;   // clusters per block of the nearest-node kernel
constexpr int kKmPad = 64;     // zero doubles after the sums: the widest chunk may read that far past row k-1
constexpr int kKmMaxK = 4096;  // the sums' partial tables are (k + 1) k words per node range
constexpr int kKmMinBlocks = 2048;
// Pivots from which the matrix form is taken: its tiles hold 64 features and 16
// clusters, so small k pay for padding.  50 passes, vector against matrix form:
// 50k nodes k = 16 1.76 / 1.95 ms, 48 2.40 / 2.34, 64 2.77 / 2.53; 1M nodes k = 3
// (38 passes) 2.44 / 4.65, 24 9.7 / 10.4, 48 19.4 / 16.8.
constexpr int kKmMatrixMinK = 48;
constexpr int kKmBatch = 4;    // passes enqueued between looks at the flag
// control words: nodes moved in the pass, no node moved (the later passes return at once), passes run
constexpr int kKmMoved = 0, kKmDone = 1, kKmPasses = 2, kKmCtl = 4;
constexpr int kKmReduceSlice = 8;  // partial tables summed per thread before one atomic add

// ST (k k doubles, then kKmPad zero doubles so that a block's last chunk
// may read past row k-1), N, and assign = -1 (no cluster yet).
__global__ void k_km_init(int n, int k, const int* __restrict__ dist, const int* __restrict__ pivots,
                          double* __restrict__ ST, double* __restrict__ N, int* __restrict__ assign) {
    const long long kk = (long long)k * k, total = kk + kKmPad + n;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < total;
         q += (long long)gridDim.x * blockDim.x) {
        if (q < kk) {
            const int j = (int)(q / k), t = (int)(q % k);
            ST[q] = (double)dist[(size_t)j * n + pivots[t]];
            if (j == 0) N[t] = 1.0;
        } else if (q < kk + kKmPad) {
            ST[q] = 0.0;
        } else {
            assign[q - kk - kKmPad] = -1;
        }
    }
}

// ||y_i||^2 as a 64-bit integer.
__global__ void k_km_norm(int n, int k, const int* __restrict__ dist, long long* __restrict__ q) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    long long s = 0;
    for (int j = 0; j < k; ++j) {
        const long long y = dist[(size_t)j * n + i];
        s += y * y;
    }
    q[i] = s;
}

// a_t = sum_j (S_tj / N_t)^2, ascending j, each quotient, square and sum
// rounded: one block per t squares 256 features at a time in parallel, one
// lane adds them in order.
// Opens a pass: also clears the new sums S2 and the count of moved nodes.
__global__ __launch_bounds__(256) void k_km_a(int k, const double* __restrict__ ST, const double* __restrict__ N,
                                              double* __restrict__ a, unsigned long long* __restrict__ S2, int* ctl) {
#pragma clang fp contract(off)
    if (ctl[kKmDone]) return;
    __shared__ double sq[256];
    const int w = (k + 1) * k;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < w; q += gridDim.x * blockDim.x) S2[q] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) ctl[kKmMoved] = 0;
    const int t = blockIdx.x;
    const double nt = N[t];
    double s = 0.0;
    for (int j0 = 0; j0 < k; j0 += 256) {
        const int j = j0 + threadIdx.x;
        if (j < k) {
            const double c = ST[(size_t)j * k + t] / nt;
            sq[threadIdx.x] = c * c;
        }
        __syncthreads();
        if (threadIdx.x == 0)
            for (int u = 0; u < min(256, k - j0); ++u) s += sq[u];
        __syncthreads();
    }
    if (threadIdx.x == 0) a[t] = s;
}

// b[c] = B_{t0+c, i} = sum_j y_ij S_{t0+c, j} for c < C (columns at or past
// k read the zero padding or the next row: finite, never used).  One
// feature's C sums are wave-uniform loads.
template <int C>
__device__ __forceinline__ void km_contract(int n, int k, int i, int t0, const int* __restrict__ dist,
                                            const double* __restrict__ ST, double (&b)[C]) {
#pragma unroll
    for (int c = 0; c < C; ++c) b[c] = 0.0;
    const int* yp = dist + i;
    const double* sp = ST + t0;
    int j = 0;
    int yn[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) yn[u] = yp[(size_t)min(u, k - 1) * n];
    for (; j + 4 <= k; j += 4) {
        double y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) y[u] = (double)yn[u];
#pragma unroll
        for (int u = 0; u < 4; ++u) yn[u] = yp[(size_t)min(j + 4 + u, k - 1) * n];  // next group, clamped in range
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double* row = sp + (size_t)(j + u) * k;
#pragma unroll
            for (int c = 0; c < C; ++c) b[c] = __builtin_fma(y[u], row[c], b[c]);
        }
    }
    for (int u = 0; j < k; ++j, ++u) {
        const double y = (double)yn[u];
        const double* row = sp + (size_t)j * k;
#pragma unroll
        for (int c = 0; c < C; ++c) b[c] = __builtin_fma(y, row[c], b[c]);
    }
}

// Assignment, one chunk of C clusters per blockIdx.y: the first t of the
// chunk with the smallest f_t(i) goes to fb/tb[chunk][i].
template <int C>
__global__ __launch_bounds__(kKmBlock) void k_km_assign(int n, int k, const int* __restrict__ dist,
                                                        const double* __restrict__ ST, const double* __restrict__ N,
                                                        const double* __restrict__ a, double* __restrict__ fb,
                                                        int* __restrict__ tb, const int* __restrict__ ctl) {
#pragma clang fp contract(off)
    if (ctl[kKmDone]) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int t0 = blockIdx.y * C;
    const int ct = min(C, k - t0);
    double b[C];
    km_contract<C>(n, k, i, t0, dist, ST, b);
    int best = t0;
    double fbest = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (c < ct) {
            const int t = t0 + c;
            const double f = a[t] - (2.0 * b[c]) / N[t];
            if (c == 0 || f < fbest) {
                best = t;
                fbest = f;
            }
        }
    }
    fb[(size_t)blockIdx.y * n + i] = fbest;
    tb[(size_t)blockIdx.y * n + i] = best;
}

// Chunks in ascending order, strict improvement only: the lowest t with the
// smallest f.  ctl counts the moved nodes.
__global__ __launch_bounds__(kKmBlock) void k_km_pick(int n, int nchunks, const double* __restrict__ fb,
                                                      const int* __restrict__ tb, int* __restrict__ assign,
                                                      int* ctl) {
    if (ctl[kKmDone]) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool moved = false;
    if (i < n) {
        double fbest = fb[i];
        int best = tb[i];
        for (int c = 1; c < nchunks; ++c) {
            const double f = fb[(size_t)c * n + i];
            if (f < fbest) {
                fbest = f;
                best = tb[(size_t)c * n + i];
            }
        }
        moved = assign[i] != best;
        assign[i] = best;
    }
    const unsigned long long m = __ballot(moved);
    if (lane_id() == 0 && m) atomicAdd(&ctl[kKmMoved], (int)__popcll(m));
}

// ------------------------------------ assignment on the 8-bit matrix units
//
// y_ij and S_tj are split into signed base-256 digits (LY and LS of them), so
// that B_ti = sum over digits a, b of 256^(a + b) sum_j y^a_ij S^b_tj, and the
// inner sums are 8-bit products added in 32 bits (k digits of at most 128 x
// 128, min(LY, LS) products per power: below 2^31 up to k = 4096).  They are
// put together in 64-bit integers, so B_ti, f_t(i) and the choice are the
// vector form's, bit for bit.  50k nodes, k = 100 (2 x 4 digits): 25 us a pass
// against 48 us of FP64 FMAs and 6 us for picking the best of their chunks; the
// products are 5 us of the matrix rate, the divisions about as long, the rest
// is reading the sums' digits from L2 (57 KB per 32 nodes).  With the passes'
// flag on the device, 50 passes take 3.2 ms instead of 5.8 ms.

typedef int v4i __attribute__((ext_vector_type(4)));

// The digits of v >= 0, least significant first, each in [-128, 127].
template <int L>
__device__ __forceinline__ void km_digits(long long v, int (&d)[L]) {
#pragma unroll
    for (int l = 0; l < L; ++l) {
        d[l] = (int)((v + 128) & 255) - 128;
        v = (v - d[l]) >> 8;
    }
}

// Digits that hold every value up to `most`.
static int km_digit_count(double most) {
    int l = 1;
    for (double top = 127.0; top < most; top = top * 256.0 + 127.0) ++l;
    return l;
}

// Y[l][j / 16][i]: the l-th digits of y_ij for 16 features of node i (zero past k).
template <int LY>
__global__ __launch_bounds__(256) void k_km_ydigits(int n, int k, int nkb, const int* __restrict__ dist,
                                                    uint4* __restrict__ Y) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, b = blockIdx.y;
    if (i >= n) return;
    int y[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) y[u] = dist[(size_t)min(16 * b + u, k - 1) * n + i];
    unsigned w[LY][4] = {};
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        int d[LY];
        km_digits<LY>(16 * b + u < k ? y[u] : 0, d);
#pragma unroll
        for (int l = 0; l < LY; ++l) w[l][u / 4] |= (unsigned)(d[l] & 255) << (8 * (u % 4));
    }
#pragma unroll
    for (int l = 0; l < LY; ++l)
        Y[((size_t)l * nkb + b) * n + i] = make_uint4(w[l][0], w[l][1], w[l][2], w[l][3]);
}

// Closes a pass (S2 not null): non-empty clusters take their new sums, an
// empty one keeps its centroid, and the pass is counted; no node moved ends
// the passes.  (A block that starts after that flag was set returns at once:
// the sums are the last pass's then.)  Also writes the sums' digits
// Sq[l][j / 16][t], t < kc (zero past k); S2 null: the digits alone.
template <int LS>
__global__ __launch_bounds__(256) void k_km_commit_mx(int k, int nkb, int kc, const unsigned long long* __restrict__ S2,
                                                      double* __restrict__ ST, double* __restrict__ N,
                                                      uint4* __restrict__ Sq, int* ctl) {
    if (ctl[kKmDone]) return;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    const int t = q % kc, b = q / kc;
    if (b < nkb) {
        const unsigned long long cnt = S2 && t < k ? S2[(size_t)k * k + t] : 0;
        long long v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int j = 16 * b + u;
            v[u] = 0;
            if (t < k && j < k) v[u] = cnt ? (long long)S2[(size_t)j * k + t] : (long long)ST[(size_t)j * k + t];
        }
        if (cnt) {
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (16 * b + u < k) ST[(size_t)(16 * b + u) * k + t] = (double)v[u];
            if (b == 0) N[t] = (double)cnt;
        }
        unsigned w[LS][4] = {};
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            int d[LS];
            km_digits<LS>(v[u], d);
#pragma unroll
            for (int l = 0; l < LS; ++l) w[l][u / 4] |= (unsigned)(d[l] & 255) << (8 * (u % 4));
        }
#pragma unroll
        for (int l = 0; l < LS; ++l)
            Sq[((size_t)l * nkb + b) * kc + t] = make_uint4(w[l][0], w[l][1], w[l][2], w[l][3]);
    }
    if (S2 && q == 0) {
        ctl[kKmPasses] += 1;
        if (ctl[kKmMoved] == 0) ctl[kKmDone] = 1;
    }
}

// Assignment of 32 nodes per wave to the nearest of all k clusters: 16 x 16
// tiles of B over the features, 64 per matrix instruction; the nodes' digits
// stay in registers for up to 128 features (KSR = 64-feature steps; 0: read
// again for every 16 clusters).  Lane (c, g) = (lane % 16, lane / 16) holds B
// of nodes 4 g .. 4 g + 3 of a tile and cluster c, keeps its best cluster in
// ascending order, and 16 lanes settle a node at the end (smallest f, lowest t).
template <int LY, int LS, int KSR>
__global__ __launch_bounds__(256) void k_km_assign_mx(int n, int k, int nkb, int kc, const uint4* __restrict__ Y,
                                                      const uint4* __restrict__ Sq, const double* __restrict__ N,
                                                      const double* __restrict__ a, int* __restrict__ assign, int* ctl) {
#pragma clang fp contract(off)
    if (ctl[kKmDone]) return;
    constexpr int MT = 2, NG = LY + LS - 1;
    const int lane = lane_id(), c16 = lane % 16, g = lane / 16;
    const int i0 = (blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave) * 16 * MT;
    if (i0 >= n) return;  // uniform per wave
    const int steps = KSR > 0 ? KSR : nkb / 4;
    auto load_y = [&](int m, int l, int ks) {
        const uint4 v = Y[((size_t)l * nkb + 4 * ks + g) * n + min(i0 + 16 * m + c16, n - 1)];
        return v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
    };
    v4i A[MT][LY][KSR > 0 ? KSR : 1];
    if (KSR > 0) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int l = 0; l < LY; ++l)
#pragma unroll
                for (int ks = 0; ks < (KSR > 0 ? KSR : 1); ++ks) A[m][l][ks] = load_y(m, l, ks);
    }
    double bf[MT][4];
    int bt[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            bf[m][r] = __builtin_inf();
            bt[m][r] = INT_MAX;
        }
    for (int t0 = 0; t0 < kc; t0 += 16) {
        v4i acc[MT][NG];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int e = 0; e < NG; ++e) acc[m][e] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < steps; ++ks) {
            v4i B[LS];
#pragma unroll
            for (int l = 0; l < LS; ++l) {
                const uint4 v = Sq[((size_t)l * nkb + 4 * ks + g) * kc + t0 + c16];
                B[l] = v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
            }
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int l = 0; l < LY; ++l) {
                    const v4i y = KSR > 0 ? A[m][l][KSR > 0 ? ks : 0] : load_y(m, l, ks);
#pragma unroll
                    for (int b = 0; b < LS; ++b)
                        acc[m][l + b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(y, B[b], acc[m][l + b], 0, 0, 0);
                }
        }
        const int t = t0 + c16;
        const double at = a[min(t, k - 1)], nt = N[min(t, k - 1)];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                long long b = 0;
#pragma unroll
                for (int e = NG - 1; e >= 0; --e) b = b * 256 + acc[m][e][r];
                const double f = at - (2.0 * (double)b) / nt;
                if (t < k && f < bf[m][r]) {
                    bf[m][r] = f;
                    bt[m][r] = t;
                }
            }
    }
    int moved = 0;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) {
                const double f = __shfl_xor(bf[m][r], off);
                const int t = __shfl_xor(bt[m][r], off);
                if (f < bf[m][r] || (f == bf[m][r] && t < bt[m][r])) {
                    bf[m][r] = f;
                    bt[m][r] = t;
                }
            }
            const int i = i0 + 16 * m + 4 * g + r;
            if (c16 == 0 && i < n && assign[i] != bt[m][r]) {
                assign[i] = bt[m][r];
                ++moved;
            }
        }
    moved = wave_sum(moved);
    if (lane == 0 && moved) atomicAdd(&ctl[kKmMoved], moved);
}

template <int LY, int LS>
static hipError_t km_assign_mx(int n, int k, int nkb, int kc, const uint4* Y, const uint4* Sq, const double* N,
                               const double* a, int* assign, int* ctl, hipStream_t s) {
    auto kern = nkb == 4 ? k_km_assign_mx<LY, LS, 1> : nkb == 8 ? k_km_assign_mx<LY, LS, 2> : k_km_assign_mx<LY, LS, 0>;
    hipLaunchKernelGGL(kern, dim3(div_up(n, 128)), dim3(256), 0, s, n, k, nkb, kc, Y, Sq, N, a, assign, ctl);
    return hipGetLastError();
}

// Built for LS in 2 .. 5.
template <int LS>
static hipError_t km_commit_mx(int k, int nkb, int kc, const unsigned long long* S2, double* ST, double* N, uint4* Sq,
                               int* ctl, hipStream_t s) {
    hipLaunchKernelGGL(k_km_commit_mx<LS>, dim3(div_up(nkb * kc, 256)), dim3(256), 0, s, k, nkb, kc, S2, ST, N, Sq, ctl);
    return hipGetLastError();
}

// Member sums of `rows` feature rows (row k = member counts) over nodes
// [bx span, (bx+1) span): LDS 64-bit counters, one add per wave when the
// whole wave shares a cluster, else one per node.  Each block writes its
// partial table part[bx][j0 .. j0+rows)[k].
__global__ __launch_bounds__(kKmBlock) void k_km_sums(int n, int k, int rows_per_block, int span,
                                                      const int* __restrict__ dist, const int* __restrict__ assign,
                                                      unsigned long long* __restrict__ part,
                                                      const int* __restrict__ ctl) {
    if (ctl[kKmDone]) return;
    extern __shared__ unsigned long long acc[];  // [rows_per_block][k]
    const int j0 = blockIdx.y * rows_per_block;
    const int rows = min(rows_per_block, k + 1 - j0);
    for (int q = threadIdx.x; q < rows * k; q += blockDim.x) acc[q] = 0;
    __syncthreads();
    const int i0 = blockIdx.x * span, i1 = min(n, i0 + span);
    for (int base = i0; base < i1; base += blockDim.x) {
        const int i = base + threadIdx.x;
        const bool ok = i < i1;
        const int t = ok ? assign[i] : 0;
        const int tf = __builtin_amdgcn_readfirstlane(t);
        const bool uniform = __ballot(!ok || t != tf) == 0;
        for (int r = 0; r < rows; ++r) {
            const int j = j0 + r;
            long long v = 0;
            if (ok) v = j < k ? (long long)dist[(size_t)j * n + i] : 1;
            if (uniform) {
                v = wave_sum(v);
                if (lane_id() == 0) atomicAdd(&acc[r * k + tf], (unsigned long long)v);
            } else if (ok) {
                atomicAdd(&acc[r * k + t], (unsigned long long)v);
            }
        }
    }
    __syncthreads();
    unsigned long long* out = part + (size_t)blockIdx.x * (k + 1) * k + (size_t)j0 * k;
    for (int q = threadIdx.x; q < rows * k; q += blockDim.x) out[q] = acc[q];
}

// S2 (zeroed) += the partial tables of blocks [y slice, (y+1) slice).
__global__ void k_km_reduce(int nbx, int slice, int k, const unsigned long long* __restrict__ part,
                            unsigned long long* __restrict__ S2, const int* __restrict__ ctl) {
    if (ctl[kKmDone]) return;
    const long long w = (long long)(k + 1) * k;
    const long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (q >= w) return;
    const int b0 = blockIdx.y * slice, b1 = min(nbx, b0 + slice);
    unsigned long long s = 0;
    for (int bx = b0; bx < b1; ++bx) s += part[(size_t)bx * w + q];
    if (s) atomicAdd(&S2[q], s);
}

// k_km_commit_mx without the digits.
__global__ void k_km_commit(int k, const unsigned long long* __restrict__ S2, double* __restrict__ ST,
                            double* __restrict__ N, int* ctl) {
    if (ctl[kKmDone]) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctl[kKmPasses] += 1;
        if (ctl[kKmMoved] == 0) ctl[kKmDone] = 1;
    }
    const long long kk = (long long)k * k;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < kk;
         q += (long long)gridDim.x * blockDim.x) {
        const int j = (int)(q / k), t = (int)(q % k);
        const unsigned long long cnt = S2[kk + t];
        if (cnt > 0) {
            ST[q] = (double)S2[q];
            if (j == 0) N[t] = (double)cnt;
        }
    }
}

__device__ __forceinline__ void km_argmin_pair(long long& s, int& id, long long s2, int id2) {
    if (s2 < s || (s2 == s && id2 < id)) {
        s = s2;
        id = id2;
    }
}

// Nearest free node to each of C centroids t_base + blockIdx.y C + c over
// this block's nodes: smallest N_t q_i - 2 B_ti, then lowest id; one
// (score, node) pair per (block, t) into ps/pn[bx][t].
template <int C>
__global__ __launch_bounds__(kKmBlock) void k_km_near(int n, int k, int t_base, const int* __restrict__ dist,
                                                      const double* __restrict__ ST, const double* __restrict__ N,
                                                      const long long* __restrict__ q,
                                                      const unsigned char* __restrict__ taken,
                                                      long long* __restrict__ ps, int* __restrict__ pn) {
    __shared__ long long ws[kKmBlock / kWave][C];
    __shared__ int wn[kKmBlock / kWave][C];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int t0 = t_base + blockIdx.y * C;
    const int ct = min(C, k - t0);
    double b[C];
    const bool live = i < n && !taken[i];
    if (i < n) km_contract<C>(n, k, i, t0, dist, ST, b);
    const long long qi = live ? q[i] : 0;
    const int w = threadIdx.x / kWave;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (c < ct) {
            long long s = LLONG_MAX;
            int id = INT_MAX;
            if (live) {
                s = (long long)N[t0 + c] * qi - 2 * (long long)b[c];
                id = i;
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) km_argmin_pair(s, id, __shfl_xor(s, off), __shfl_xor(id, off));
            if (lane_id() == 0) {
                ws[w][c] = s;
                wn[w][c] = id;
            }
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < ct) {
        const int c = threadIdx.x;
        long long s = ws[0][c];
        int id = wn[0][c];
        for (int u = 1; u < kKmBlock / kWave; ++u) km_argmin_pair(s, id, ws[u][c], wn[u][c]);
        ps[(size_t)blockIdx.x * k + t0 + c] = s;
        pn[(size_t)blockIdx.x * k + t0 + c] = id;
    }
}

// One block per t: the (score, node) minimum over the nbx block results.
__global__ __launch_bounds__(256) void k_km_near_reduce(int nbx, int k, int t_base, const long long* __restrict__ ps,
                                                        const int* __restrict__ pn, int* __restrict__ node) {
    __shared__ long long ws[256 / kWave];
    __shared__ int wn[256 / kWave];
    const int t = t_base + blockIdx.x;
    long long s = LLONG_MAX;
    int id = INT_MAX;
    for (int bx = threadIdx.x; bx < nbx; bx += blockDim.x)
        km_argmin_pair(s, id, ps[(size_t)bx * k + t], pn[(size_t)bx * k + t]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) km_argmin_pair(s, id, __shfl_xor(s, off), __shfl_xor(id, off));
    if (lane_id() == 0) {
        ws[threadIdx.x / kWave] = s;
        wn[threadIdx.x / kWave] = id;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int u = 1; u < 256 / kWave; ++u) km_argmin_pair(s, id, ws[u], wn[u]);
        node[t] = id == INT_MAX ? -1 : id;
    }
}

// Largest entry of dist (block maxima, one atomic per block).
__global__ __launch_bounds__(256) void k_km_dmax(long long total, const int* __restrict__ dist, int* out) {
    int m = 0;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < total;
         q += (long long)gridDim.x * blockDim.x)
        m = max(m, dist[q]);
    __shared__ int red[256 / kWave];
    m = block_max(m, red);
    if (threadIdx.x == 0) atomicMax(out, m);
}

namespace {

hipError_t km_nearest(int n, int k, int t_base, int t_count, const int* dist, const double* ST, const double* N,
                      const long long* q, const unsigned char* taken, long long* ps, int* pn, int* node,
                      hipStream_t s) {
    const int nb = div_up(n, kKmBlock);
    if (t_count == 1) {
        hipLaunchKernelGGL(k_km_near<1>, dim3(nb, 1), dim3(kKmBlock), 0, s, n, k, t_base, dist, ST, N, q, taken, ps,
                           pn);
    } else {
        hipLaunchKernelGGL(k_km_near<kKmChunk>, dim3(nb, div_up(t_count, kKmChunk)), dim3(kKmBlock), 0, s, n, k,
                           t_base, dist, ST, N, q, taken, ps, pn);
    }
    hipLaunchKernelGGL(k_km_near_reduce, dim3(t_count), dim3(256), 0, s, nb, k, t_base, ps, pn, node);
    return hipGetLastError();
}

}  // namespace

ssm_status kmeans_pivots(int32_t n, int32_t k, const int32_t* pivots, const int32_t* dist, int32_t max_iters,
                         int32_t* new_pivots, int32_t* assign_out, int32_t* iters_host, hipStream_t s) {
    if (k > kKmMaxK) return fail(SSM_E_RANGE, "k-means sp: k above 4096");
    {  // the pivots index the distance rows' columns
        std::vector<int> hp(k);
        hipError_t e0 = hipMemcpyAsync(hp.data(), pivots, sizeof(int) * k, hipMemcpyDeviceToHost, s);
        if (e0 == hipSuccess) e0 = hipStreamSynchronize(s);
        if (e0 != hipSuccess) return hip_fail(e0, "k-means sp: pivots");
        for (int t = 0; t < k; ++t)
            if (hp[t] < 0 || hp[t] >= n) return fail(SSM_E_INVAL, "k-means sp: pivot out of range");
    }
    int dmax = 0;
    {  // every product and sum of the exact integer arithmetic stays below 2^53
        int* dm = nullptr;
        ssm_status st0 = salloc((void**)&dm, sizeof(int));
        if (st0 != SSM_OK) return st0;
        int hdm = 0;
        hipError_t e0 = hipMemsetAsync(dm, 0, sizeof(int), s);
        if (e0 == hipSuccess) {
            hipLaunchKernelGGL(k_km_dmax, dim3(std::max(1, std::min(div_up((long long)k * n, 256), 4096))), dim3(256),
                               0, s, (long long)k * n, dist, dm);
            e0 = hipGetLastError();
        }
        if (e0 == hipSuccess) e0 = hipMemcpyAsync(&hdm, dm, sizeof(int), hipMemcpyDeviceToHost, s);
        if (e0 == hipSuccess) e0 = hipStreamSynchronize(s);
        (void)hipStreamSynchronize(s);
        sfree(dm);
        if (e0 != hipSuccess) return hip_fail(e0, "k-means sp: distance range");
        if ((double)k * (double)n * (double)hdm * (double)hdm >= 9007199254740992.0)
            return fail(SSM_E_RANGE, "k-means sp: k * n * dmax^2 reaches 2^53 (exact integer sums not guaranteed)");
        dmax = hdm;
    }
    // the matrix form's digits; other counts (distances above 32,639, sums
    // above 5.4e11) take the vector form, as does a forced km_chunk (tuning:
    // km_matrix -1 = never, 1 = whatever k)
    const int ly = km_digit_count(dmax), ls = std::max(2, km_digit_count((double)n * dmax));
    const int forced = variant("km_matrix");
    bool mx = ly <= 2 && ls <= 5 && variant("km_chunk") == 0 && forced >= 0 && (forced == 1 || k >= kKmMatrixMinK);
    const int nkb = div_up(k, 64) * 4, kc = div_up(k, 16) * 16;
    // launch shapes
    const int nb = div_up(n, kKmBlock);
    // assignment chunk: fewest padded clusters, each chunk costing about 8
    // more for its re-read of the distance table
    int C = 0, cost = INT_MAX;
    for (int c : {32, 40, 48, 56, 64}) {
        const int cc = div_up(k, c) * (c + 8);
        if (cc < cost) {
            cost = cc;
            C = c;
        }
    }
    if (const int c = variant("km_chunk")) {
        if (c == 32 || c == 40 || c == 48 || c == 56 || c == 64) C = c;
    }
    const int nchunks = div_up(k, C);
    auto assign_kernel = C == 32 ? k_km_assign<32> : C == 40 ? k_km_assign<40> : C == 48 ? k_km_assign<48>
                       : C == 56 ? k_km_assign<56> : k_km_assign<64>;
    const int rows_per_block = std::max(1, std::min(8, 4096 / k));  // LDS: rows k 8 bytes <= 32 KB
    const int ny = div_up(k + 1, rows_per_block);
    int nbx = std::max(1, std::min(nb, div_up(kKmMinBlocks, ny)));
    const int span = div_up(div_up(n, nbx), kKmBlock) * kKmBlock;
    nbx = div_up(n, span);
    // workspace
    const size_t kk = (size_t)k * k, w = (size_t)(k + 1) * k;
    size_t off = 0, o_st, o_n, o_a, o_q, o_fb, o_tb, o_as, o_ch,
           o_y, o_sq, o_part, o_s2, o_ps, o_pn, o_tk, o_nd;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    auto lay_out = [&] {
        off = 0;
        o_st = take(sizeof(double) * (kk + kKmPad));
        o_n = take(sizeof(double) * k);
        o_a = take(sizeof(double) * k);
        o_q = take(sizeof(long long) * n);
        o_fb = take(mx ? 0 : sizeof(double) * (size_t)nchunks * n);
        o_tb = take(mx ? 0 : sizeof(int) * (size_t)nchunks * n);
        o_as = take(sizeof(int) * (size_t)n);
        o_ch = take(sizeof(int) * kKmCtl);
        o_y = take(mx ? sizeof(uint4) * (size_t)ly * nkb * n : 0);
        o_sq = take(mx ? sizeof(uint4) * (size_t)ls * nkb * kc : 0);
        o_part = take(sizeof(unsigned long long) * (size_t)nbx * w);
        o_s2 = take(sizeof(unsigned long long) * w);
        o_ps = take(sizeof(long long) * (size_t)nb * k);
        o_pn = take(sizeof(int) * (size_t)nb * k);
        o_tk = take((size_t)n);
        o_nd = take(sizeof(int) * k);
    };
    lay_out();
    char* ws = nullptr;
    ssm_status st = salloc((void**)&ws, off);
    if (st == SSM_E_NOMEM && mx) {  // the matrix form also holds the table's digits
        mx = false;
        lay_out();
        st = salloc((void**)&ws, off);
    }
    if (st != SSM_OK) return st;
    double* ST = (double*)(ws + o_st);
    double* N = (double*)(ws + o_n);
    double* a = (double*)(ws + o_a);
    long long* q = (long long*)(ws + o_q);
    double* fb = (double*)(ws + o_fb);
    int* tb = (int*)(ws + o_tb);
    int* assign = assign_out ? assign_out : (int*)(ws + o_as);
    int* ctl = (int*)(ws + o_ch);
    uint4* Y = (uint4*)(ws + o_y);
    uint4* Sq = (uint4*)(ws + o_sq);
    unsigned long long* part = (unsigned long long*)(ws + o_part);
    unsigned long long* S2 = (unsigned long long*)(ws + o_s2);
    long long* ps = (long long*)(ws + o_ps);
    int* pn = (int*)(ws + o_pn);
    unsigned char* taken = (unsigned char*)(ws + o_tk);
    int* nodes = (int*)(ws + o_nd);

    const int grid_init = std::max(1, std::min(div_up((long long)kk + kKmPad + n, 256), 8192));
    hipLaunchKernelGGL(k_km_init, dim3(grid_init), dim3(256), 0, s, n, k, dist, pivots, ST, N, assign);
    hipLaunchKernelGGL(k_km_norm, dim3(nb), dim3(kKmBlock), 0, s, n, k, dist, q);
    hipError_t e = hipMemsetAsync(ctl, 0, sizeof(int) * kKmCtl, s);
    if (e == hipSuccess) e = hipGetLastError();
    auto commit = [&](const unsigned long long* sums) {
        switch (ls) {
            case 2: return km_commit_mx<2>(k, nkb, kc, sums, ST, N, Sq, ctl, s);
            case 3: return km_commit_mx<3>(k, nkb, kc, sums, ST, N, Sq, ctl, s);
            case 4: return km_commit_mx<4>(k, nkb, kc, sums, ST, N, Sq, ctl, s);
            default: return km_commit_mx<5>(k, nkb, kc, sums, ST, N, Sq, ctl, s);
        }
    };
    auto assign_mx = [&]() {
#define SSM_KM(LS_)                                                                                  \
    return ly == 1 ? km_assign_mx<1, LS_>(n, k, nkb, kc, Y, Sq, N, a, assign, ctl, s)                \
                   : km_assign_mx<2, LS_>(n, k, nkb, kc, Y, Sq, N, a, assign, ctl, s)
        switch (ls) {
            case 2: SSM_KM(2);
            case 3: SSM_KM(3);
            case 4: SSM_KM(4);
            default: SSM_KM(5);
        }
#undef SSM_KM
    };
    if (mx && e == hipSuccess) {
        hipLaunchKernelGGL(ly == 1 ? k_km_ydigits<1> : k_km_ydigits<2>, dim3(nb, nkb), dim3(kKmBlock), 0, s, n, k, nkb,
                           dist, Y);
        e = commit(nullptr);
    }
    int it = 0;
    for (int queued = 0; e == hipSuccess && queued < max_iters;) {
        for (int b = 0; b < kKmBatch && queued < max_iters && e == hipSuccess; ++b, ++queued) {
            hipLaunchKernelGGL(k_km_a, dim3(k), dim3(256), 0, s, k, ST, N, a, S2, ctl);
            if (mx) {
                e = assign_mx();
            } else {
                hipLaunchKernelGGL(assign_kernel, dim3(nb, nchunks), dim3(kKmBlock), 0, s, n, k, dist, ST, N, a, fb, tb,
                                   ctl);
                hipLaunchKernelGGL(k_km_pick, dim3(nb), dim3(kKmBlock), 0, s, n, nchunks, fb, tb, assign, ctl);
            }
            hipLaunchKernelGGL(k_km_sums, dim3(nbx, ny), dim3(kKmBlock),
                               sizeof(unsigned long long) * (size_t)rows_per_block * k, s, n, k, rows_per_block, span,
                               dist, assign, part, ctl);
            hipLaunchKernelGGL(k_km_reduce, dim3(div_up((long long)w, 256), div_up(nbx, kKmReduceSlice)), dim3(256), 0,
                               s, nbx, kKmReduceSlice, k, part, S2, ctl);
            if (mx)
                e = e == hipSuccess ? commit(S2) : e;
            else
                hipLaunchKernelGGL(k_km_commit, dim3(std::max(1, std::min(div_up((long long)kk, 256), 4096))), dim3(256),
                                   0, s, k, S2, ST, N, ctl);
            if (e == hipSuccess) e = hipGetLastError();
        }
        int h[kKmCtl] = {};
        if (e == hipSuccess) e = hipMemcpyAsync(h, ctl, sizeof h, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        it = h[kKmPasses];
        if (h[kKmDone]) break;
    }
    // nearest free node per cluster: all clusters at once, then each one
    // whose choice a lower rank already took again, without the taken nodes
    std::vector<int> hnodes(k);
    if (e == hipSuccess) e = hipMemsetAsync(taken, 0, (size_t)n, s);
    if (e == hipSuccess) e = km_nearest(n, k, 0, k, dist, ST, N, q, taken, ps, pn, nodes, s);
    if (e == hipSuccess) e = hipMemcpyAsync(hnodes.data(), nodes, sizeof(int) * k, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    std::vector<int> result(k, -1);
    std::vector<unsigned char> used;
    if (e == hipSuccess) used.assign((size_t)n, 0);
    for (int t = 0; t < k && e == hipSuccess; ++t) {
        int v = hnodes[t];
        if (v < 0 || used[v]) {
            e = hipMemcpyAsync(taken, used.data(), (size_t)n, hipMemcpyHostToDevice, s);
            if (e == hipSuccess) e = km_nearest(n, k, t, 1, dist, ST, N, q, taken, ps, pn, nodes, s);
            if (e == hipSuccess) e = hipMemcpyAsync(&v, nodes + t, sizeof(int), hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e != hipSuccess) break;
            if (v < 0) {  // cannot happen: fewer than k nodes are taken
                e = hipErrorUnknown;
                break;
            }
        }
        result[t] = v;
        used[v] = 1;
    }
    if (e == hipSuccess) e = hipMemcpyAsync(new_pivots, result.data(), sizeof(int) * k, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipStreamSynchronize(s);
    sfree(ws);
    if (e != hipSuccess) return hip_fail(e, "k-means sp");
    if (iters_host) *iters_host = it;
    return SSM_OK;
}

}  // namespace ssm
