// Frozen-core folding of the folded operator (the xTC-FC scheme of the
// results section: corrections computed with all electrons, then the standard
// closed-shell frozen-core equations), with V2[p][q][r][s] = (pq|rs):
//   E  = E0 + 2 sum_c h1[c][c] + sum_{c,d} (2 (cc|dd) - (cd|dc))
//   h[i][j] = h1[a_i][a_j] + sum_c (2 (a_i a_j|cc) - (a_i c|c a_j))
//   V[i][j][k][l] = V2[a_i][a_j][a_k][a_l]
// Every element of h is one thread's fixed-order sum, E one workgroup's sum by a
// fixed tree (deterministic).
#pragma once
#include "xtc_device.h"

namespace xtc {

constexpr int kMaxFcList = 256;
struct IdxList {
    int32_t n;
    int32_t k[kMaxFcList];
};

// One launch: workgroup 0 takes E, the next n_h h, and the rest one (i, j) row
// each of V (na^2 values of V2's row (a_i, a_j), read in runs of consecutive
// active orbitals).  Bound by V's copy: N=96, 84 active 290 -> 168 us (three
// launches one after the other before, E by a single thread in 71 us).
__global__ __launch_bounds__(256) void k_frozen_core(const double* __restrict__ V2, const double* __restrict__ h1,
                                                     const double* __restrict__ E0, int N, IdxList core, IdxList act,
                                                     int n_h, double* __restrict__ V, double* __restrict__ h,
                                                     double* __restrict__ E) {
    const size_t n = (size_t)N;
    const int na = act.n, nc = core.n;
    if (blockIdx.x == 0) {
        double e = 0.0;
        for (int ci = threadIdx.x; ci < nc; ci += 256) e += 2.0 * h1[core.k[ci] * n + core.k[ci]];
        for (int cd = threadIdx.x; cd < nc * nc; cd += 256) {
            const int c = core.k[cd / nc], d = core.k[cd % nc];
            e += 2.0 * V2[((c * n + c) * n + d) * n + d] - V2[((c * n + d) * n + d) * n + c];
        }
        __shared__ double red[256];
        red[threadIdx.x] = e;
        __syncthreads();
        for (int m = 128; m >= 1; m >>= 1) {
            if ((int)threadIdx.x < m) red[threadIdx.x] += red[threadIdx.x + m];
            __syncthreads();
        }
        if (threadIdx.x == 0) *E = *E0 + red[0];
        return;
    }
    if ((int)blockIdx.x <= n_h) {
        const int ij = (blockIdx.x - 1) * 256 + threadIdx.x;
        if (ij >= na * na) return;
        const int p = act.k[ij / na], q = act.k[ij % na];
        double v = h1[p * n + q];
        for (int cc = 0; cc < nc; ++cc) {
            const int c = core.k[cc];
            v += 2.0 * V2[((p * n + q) * n + c) * n + c] - V2[((p * n + c) * n + c) * n + q];
        }
        h[ij] = v;
        return;
    }
    const int ij = blockIdx.x - 1 - n_h;
    const double* src = V2 + ((size_t)act.k[ij / na] * n + act.k[ij % na]) * n * n;
    double* dst = V + (size_t)ij * na * na;
    __shared__ int list[kMaxFcList];
    for (int i = threadIdx.x; i < na; i += 256) list[i] = act.k[i];
    __syncthreads();
    constexpr int kAhead = 8;
    for (int t0 = threadIdx.x; t0 < na * na; t0 += 256 * kAhead) {
        double v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int t = min(t0 + 256 * u, na * na - 1);
            v[u] = src[(size_t)list[t / na] * n + list[t % na]];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (t0 + 256 * u < na * na) dst[t0 + 256 * u] = v[u];
    }
}

}  // namespace xtc
