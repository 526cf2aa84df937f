// Grid intermediate K^x_P(g) = sum_g' d^x(g,g') rho_P(g')  (FP64 MFMA).
//
// The sum over g' is a GEMM whose left operand d^x(g,g') is generated on chip
// from the grid positions (never stored: Ng^2 values) and whose right operand
// is the prepared weighted pair density rho[g'][P] (all pairs, or the gathered
// occupied ones of the reduced forms).  One MFMA v_mfma_f64_16x16x4_f64
// consumes a 16(g) x 4(g') slab of d^x and a 4(g') x 16(P) slab of rho.
//
// Operand layouts of v_mfma_f64_16x16x4_f64 (64 lanes, lane l):
//   A[i][k]: i = l % 16, k = l / 16      B[k][j]: k = l / 16, j = l % 16
//   D[i][j]: lane l holds rows i = l/16 + 4 v, v = 0..3, column j = l % 16
//   (decoded on gfx950; it differs from the FP32 form's 4 (l/16) + v).
#pragma once
#include "xtc_device.h"

namespace xtc {

constexpr int kKSteps = 8;                  // 4-point k-steps per stage
constexpr int kKStage = 4 * kKSteps;        // grid points per stage
constexpr int kKSegQuant = 2 * kKStage;     // segments are whole pairs of stages

// Workgroup: 4 waves as 4/CW (16-row groups) x CW (column groups of 16 NB);
// each wave owns 16 rows and the 3 vector components of its columns (3 NB
// accumulator blocks).  The CW waves of a row group share its d^x: each
// generates kKSteps / CW of the next stage's k-steps (one value of each
// component per lane) into one of two LDS buffers while the current stage is
// multiplied, one barrier per stage.
// Why shared: FP64 VALU instructions and FP64 MFMA do not overlap (the MFMA
// pipes were busy 0.805 of the cycles with 46 VALU instructions per 24 MFMAs,
// as if each VALU instruction held them for 8 cycles), so what a wave does not
// generate is time.  kDepth k-steps of rho are in flight in registers.
// N=64, 20 000 points: 85.9 -> 72.7 ms, 68.7 TFLOP/s of the 78.6 peak (each
// wave generating for its own 128 columns before); N=24, 4001 points (power
// Jastrow) 926 -> 490 us, N=8, 2000 points 417 -> 35 us (in segments, and
// narrower columns).  The 210 occupied pairs of N=64, 5000 rows: 2626 -> 2451
// us against the kernel that staged rho in LDS and generated per wave.
// Within a wave's columns, block c of a group of VW blocks maps logical column
// j to VW j + c, so that a lane loads and stores VW consecutive values.
// blockIdx.x: row tile fastest, so workgroups resident at the same time share
// one column strip of rho through L2; blockIdx.y: segment of seg_len points.
template <int KIND, int NB, int CW>
__global__ __launch_bounds__(256, 1) void k_build_K_f64(const d4* __restrict__ pos,
                                                                     const double* __restrict__ rho, int ld, int ngp,
                                                                     int g0, int rows, int n_rt, int seg_len,
                                                                     JasDev J, double* __restrict__ out, int ldo,
                                                                     int ncol) {
    constexpr int kRows = 16 * (4 / CW);                 // grid rows per workgroup
    constexpr int kGen = kKSteps / CW;                   // k-steps a wave generates per stage
    constexpr int VW = NB % 4 == 0 ? 4 : NB % 2 == 0 ? 2 : 1;
    constexpr int kDepth = NB >= 5 ? 2 : 4;
    typedef double vec __attribute__((ext_vector_type(VW)));
    typedef double ATile[4 / CW][kKSteps][3][64];
    __shared__ ATile sA0;
    __shared__ ATile sA1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = wave / CW, cg = wave % CW;
    const int rt = blockIdx.x % n_rt, ct = blockIdx.x / n_rt;
    const int gs = blockIdx.y * seg_len, ge = min(ngp, gs + seg_len);
    const int nst = (ge - gs) / kKStage;
    const int rloc0 = rt * kRows + 16 * rg;              // first local row of this wave
    const int kq = lane >> 4, l16 = lane & 15;
    const d4 pg = pos[g0 + min(rloc0 + l16, rows - 1)];  // row whose d^x this lane generates
    const int col0 = (ct * CW + cg) * 16 * NB;

    d4 acc[3][NB];
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int c = 0; c < NB; ++c) acc[x][c] = (d4){0.0, 0.0, 0.0, 0.0};

    // rho: a uniform base per k-step plus a fixed lane offset (bytes)
    const uint32_t b_off = (uint32_t)(((size_t)kq * ld + VW * l16) * sizeof(double));
    vec b[kDepth][NB / VW];
    auto load_b = [&](int d, int kk) {
        const char* ub = (const char*)(rho + (size_t)min(kk, ge - 4) * ld + col0);
#pragma unroll
        for (int q = 0; q < NB / VW; ++q) b[d][q] = *(const vec*)(ub + b_off + 128 * VW * q);
    };
    double px[kGen], py[kGen], pz[kGen];
    auto load_p = [&](int j, int st) {
        const double* p = (const double*)(pos + min(gs + kKStage * st, ge - kKStage) + 4 * (j * CW + cg) + kq);
        px[j] = p[0];
        py[j] = p[1];
        pz[j] = p[2];
    };
    auto gen = [&](int j, ATile& W) {
        const double dx = pg.x - px[j], dy = pg.y - py[j], dz = pg.z - pz[j];
        const double f = du_over_r_f64<KIND>(fma(dx, dx, fma(dy, dy, dz * dz)), J);
        double* w = &W[rg][j * CW + cg][0][lane];
        w[0] = dx * f;
        w[64] = dy * f;
        w[128] = dz * f;
    };
    // one stage from tile R: its 8 k-steps, with the next stage's d^x
    // generated into W and the positions of the one after that loaded
    auto stage = [&](int st, const ATile& R, ATile& W) {
        const int k0 = gs + kKStage * st;
        double ax = R[rg][0][0][lane], ay = R[rg][0][1][lane], az = R[rg][0][2][lane];
#pragma unroll
        for (int t = 0; t < kKSteps; ++t) {
            const int d = t % kDepth;
            vec cb[NB / VW];
#pragma unroll
            for (int q = 0; q < NB / VW; ++q) cb[q] = b[d][q];
            load_b(d, k0 + 4 * (t + kDepth));
            double nx = 0.0, ny = 0.0, nz = 0.0;
            if (t + 1 < kKSteps) {
                nx = R[rg][t + 1][0][lane];
                ny = R[rg][t + 1][1][lane];
                nz = R[rg][t + 1][2][lane];
            }
            if (t < kGen) {
                gen(t, W);
                load_p(t, st + 2);
            }
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                double v;
                if constexpr (VW == 1) v = cb[c][0];
                else v = cb[c / VW][c % VW];
                acc[0][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax, v, acc[0][c], 0, 0, 0);
                acc[1][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(ay, v, acc[1][c], 0, 0, 0);
                acc[2][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(az, v, acc[2][c], 0, 0, 0);
            }
            ax = nx;
            ay = ny;
            az = nz;
        }
        __syncthreads();
    };
    for (int d = 0; d < kDepth; ++d) load_b(d, gs + 4 * d);
#pragma unroll
    for (int j = 0; j < kGen; ++j) load_p(j, 0);
#pragma unroll
    for (int j = 0; j < kGen; ++j) gen(j, sA0);
#pragma unroll
    for (int j = 0; j < kGen; ++j) load_p(j, 1);
    __syncthreads();
    // (past the last stage the last one is generated again into a buffer that
    // is never read: no branch in the stage)
    for (int st = 0; st < nst; st += 2) {
        stage(st, sA0, sA1);
        stage(st + 1, sA1, sA0);
    }

    double* o = out + (size_t)blockIdx.y * 3 * rows * ldo;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = rloc0 + kq + 4 * v;
        if (r < rows) {
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                double* row = o + ((size_t)x * rows + r) * ldo;
#pragma unroll
                for (int q = 0; q < NB / VW; ++q) {
                    vec val;
#pragma unroll
                    for (int e = 0; e < VW; ++e) val[e] = acc[x][VW * q + e][v];
                    *(vec*)(row + col0 + 16 * VW * q + VW * l16) = val;
                }
                if (col0 + 16 * NB == ncol)               // padding columns
                    for (int c = ncol + l16; c < ldo; c += 16) row[c] = 0.0;
            }
        }
    }
}

}  // namespace xtc
