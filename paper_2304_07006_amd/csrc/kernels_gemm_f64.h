// Transposed products over grid rows in FP64 (the two-body assembly and the
// contractions of the TC integrals):
//   M[i][j] (+)= sum_c sum_{g < rows} A_c[g][i] B_c[g][j]
// on v_mfma_f64_16x16x4 (64 cycles each), with A_c and B_c row-major.
#pragma once
#include "xtc_device.h"

namespace xtc {

// One component's operand: A_0 at p0, A_c at p1 + (c - 1) stride for c >= 1.
struct TnOperand {
    const double* p0;
    const double* p1;
    size_t stride;
    int ld;
};

// Each wave multiplies 64 x 64 (4 x 4 MFMA blocks): block b of a wave maps
// its logical row i to I0 + 4 i + b (and likewise for columns), so every lane
// loads one 32-byte vector of each operand per 4-row k-step.  The k-steps of
// all components run as one sequence, kTnDepth of them in flight in registers.
// Bound by the matrix cores, and near full load by power: N=64 (2080^2 outputs,
// 20 000 rows, four components) takes 12.7 ms in five row segments, 54 TFLOP/s,
// the MFMA pipes busy 0.86 of the cycles at 2.26 GHz; in one piece with one step
// in flight it took 26.4 ms, 289 tiles filling 256 CUs 1.1 times and the waves
// waiting half of their cycles.  N=24 on 4001 rows: 3250 -> 74 us, N=8 on 2000
// rows: 1565 -> 11 us (+ 10 us for the sum over segments).
//  SPLIT = 1: workgroup tile 128 x 128, the four waves as 2 x 2.
//  SPLIT = 4: workgroup tile 64 x 64, wave w taking the k-steps w, w + 4, ...
//   of the workgroup's rows; the four sums meet in LDS in a fixed order.
// blockIdx.y is a segment of seg_rows grid rows.  With one segment the tile is
// written (or added) to out; with several, segment s writes out + s part_stride
// and k_reduce_M_f64 sums them.  Rows past the end count as zero.
constexpr int kTnDepth = 4;
template <int SPLIT>
__global__ __launch_bounds__(256, 2) void k_gemm_tn_f64(TnOperand A, TnOperand B, int ncomp, int rows, int n_it,
                                                        int seg_rows, double* __restrict__ out, int ldm,
                                                        size_t part_stride, int accumulate) {
    static_assert(SPLIT == 1 || SPLIT == 4, "the four waves share a tile's area or its k range");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int it = blockIdx.x % n_it, jt = blockIdx.x / n_it;
    constexpr int kTile = SPLIT == 1 ? 128 : 64;
    const int I0 = it * kTile + (SPLIT == 1 ? 64 * (wave & 1) : 0);
    const int J0 = jt * kTile + (SPLIT == 1 ? 64 * (wave >> 1) : 0);
    const int kq = lane >> 4, l16 = lane & 15;
    const int gs = blockIdx.y * seg_rows, ge = min(rows, gs + seg_rows);
    const int first = gs + (SPLIT == 1 ? 0 : 4 * wave);
    const int total = first < ge ? ncomp * ((ge - first + 4 * SPLIT - 1) / (4 * SPLIT)) : 0;

    // the next k-step to load: component, first row, operand bases
    int comp = 0, g = first, left = total;
    const size_t ia = I0 + 4 * l16, jb = J0 + 4 * l16;
    const double* ap = A.p0 + ia;
    const double* bp = B.p0 + jb;
    struct Step {
        d4 a, b;
        bool on;
    };
    Step st[kTnDepth];
    auto load = [&](Step& s) {
        const int r = min(g + kq, ge - 1);      // rows past the end: any valid row, switched off by `on`
        s.on = left > 0 && g + kq < ge;
        s.a = *(const d4*)(ap + (size_t)r * A.ld);
        s.b = *(const d4*)(bp + (size_t)r * B.ld);
        --left;
        g += 4 * SPLIT;
        if (g >= ge) {
            g = first;
            if (comp + 1 < ncomp) {
                ++comp;
                ap = A.p1 + (comp - 1) * A.stride + ia;
                bp = B.p1 + (comp - 1) * B.stride + jb;
            }
        }
    };
    d4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = (d4){0.0, 0.0, 0.0, 0.0};
    if (total > 0) {
#pragma unroll
        for (int d = 0; d < kTnDepth; ++d) load(st[d]);
    }
    const d4 zero = {0.0, 0.0, 0.0, 0.0};
    for (int q = 0; q < total; q += kTnDepth) {
#pragma unroll
        for (int d = 0; d < kTnDepth; ++d) {
            const d4 a = st[d].on ? st[d].a : zero;
            const d4 b = st[d].on ? st[d].b : zero;
            load(st[d]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    if constexpr (SPLIT == 4) {
        // waves 2, 3 onto 0, 1, then 1 onto 0
        __shared__ double red[2][64][64];       // [wave & 1][register][lane]
#pragma unroll
        for (int step = 2; step >= 1; step >>= 1) {
            if (wave >= step && wave < 2 * step)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v) red[wave - step][16 * i + 4 * j + v][lane] = acc[i][j][v];
            __syncthreads();
            if (wave < step)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[i][j][v] += red[wave][16 * i + 4 * j + v][lane];
            __syncthreads();
        }
        if (wave != 0) return;
    }
    double* M = out + (size_t)blockIdx.y * part_stride;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int I = I0 + 4 * kq + 16 * v + i;        // logical row l/16 + 4v
            d4* o = (d4*)(M + (size_t)I * ldm + J0 + 4 * l16);
            d4 val = {acc[i][0][v], acc[i][1][v], acc[i][2][v], acc[i][3][v]};
            if (accumulate) val += *o;
            *o = val;
        }
}

// M[i][j] (+)= sum_s part[s][i][j] (fixed order), i < imax, j < jmax (a
// multiple of 4); part[s] has M's leading dimension.
__global__ void k_reduce_M_f64(const double* __restrict__ part, int nseg, size_t stride, int ldm, int imax, int jmax,
                               double* __restrict__ M, int accumulate) {
    const size_t n4 = (size_t)imax * (jmax / 4);
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n4; t += (size_t)gridDim.x * blockDim.x) {
        const size_t o = t / (jmax / 4) * ldm + t % (jmax / 4) * 4;
        d4 s = *(const d4*)(part + o);
        int q = 1;
        for (; q + 8 <= nseg; q += 8) {         // eight loads in flight, added in order
            d4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *(const d4*)(part + (q + u) * stride + o);
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; q < nseg; ++q) s += *(const d4*)(part + q * stride + o);
        d4* m = (d4*)(M + o);
        *m = accumulate ? *m + s : s;
    }
}

// K[x][r][P] = sum_s part[s][x][r][P] (fixed order) for P < ldo (a multiple
// of 4), 0 for ldo <= P < ldP.
__global__ void k_reduce_K_f64(const double* __restrict__ part, int nseg, int rows, int ldo, int ldP,
                               double* __restrict__ K) {
    const size_t n4 = (size_t)3 * rows * (ldP / 4);
    const size_t stride = (size_t)3 * rows * ldo;
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n4; t += (size_t)gridDim.x * blockDim.x) {
        const int P = (int)(t % (ldP / 4)) * 4;
        const size_t xr = t / (ldP / 4);
        d4 s = {0.0, 0.0, 0.0, 0.0};
        if (P < ldo) {
            const double* p = part + xr * ldo + P;
#pragma unroll 4
            for (int q = 0; q < nseg; ++q) s += *(const d4*)(p + q * stride);
        }
        *(d4*)(K + xr * ldP + P) = s;
    }
}

}  // namespace xtc
