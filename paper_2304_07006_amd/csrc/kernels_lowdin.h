// Symmetric (Loewdin) orthonormalisation of tabulated functions under the
// grid weights, in FP64:  S = chi diag(w) chi^T,  phi = S^{-1/2} chi.
//
// S^{-1/2} comes from a cyclic Jacobi eigen-decomposition (parallel
// round-robin ordering), which keeps the small eigenvalues of an
// ill-conditioned positive definite S to high relative accuracy.
#pragma once
#include "xtc_device.h"

namespace xtc {

// S partials: part[seg][i][j] = sum_{g in seg} w_g chi_i(g) chi_j(g) for i, j < ldS,
// in the 64 x 64 tiles on and above the diagonal.  The segments are short enough
// that their tiles fill the chip (lowdin_layout): N=128, 150 000 points in 37
// segments of all four tiles took 684 us.
// FP64 MFMA, workgroup 4 waves as 2 x 2, wave tile 32 x 32; each lane loads 4
// consecutive grid points of one row (k permuted as 4 (l/16) + e for both operands).
__global__ __launch_bounds__(256) void k_syrk_w_part(const double* __restrict__ chi, const double* __restrict__ w,
                                                     int N, int Ng, int ldS, int n_t, int seg_len,
                                                     double* __restrict__ part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int it, jt;
    pair_split(blockIdx.x, n_t, it, jt);
    const int seg = blockIdx.y;
    const int i0 = it * 64 + 32 * (wave & 1), j0 = jt * 64 + 32 * (wave >> 1);
    const int l16 = lane & 15, kq = 4 * (lane >> 4);
    const int gs = seg * seg_len, ge = min(Ng, gs + seg_len);
    d4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = (d4){0.0, 0.0, 0.0, 0.0};
    int ri[2], rj[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        ri[a] = min(i0 + 16 * a + l16, N - 1);
        rj[a] = min(j0 + 16 * a + l16, N - 1);
    }
    for (int g = gs; g < ge; g += 16) {
        double wv[4];
        double xa[2][4], xb[2][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int gg = g + kq + e;
            const bool ok = gg < ge;
            wv[e] = ok ? w[gg] : 0.0;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                xa[a][e] = ok ? chi[(size_t)ri[a] * Ng + gg] * wv[e] : 0.0;
                xb[a][e] = ok ? chi[(size_t)rj[a] * Ng + gg] : 0.0;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[a][e], xb[b][e], acc[a][b], 0, 0, 0);
    }
    double* out = part + (size_t)seg * ldS * ldS;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + 16 * a + (lane >> 4) + 4 * v;
#pragma unroll
            for (int b = 0; b < 2; ++b) out[(size_t)i * ldS + j0 + 16 * b + l16] = acc[a][b][v];
        }
}

// S[i][j] = S[j][i] = sum_seg part[seg][min][max] (fixed order, exactly symmetric).
__global__ void k_syrk_reduce(const double* __restrict__ part, int nseg, int N, int ldS, double* __restrict__ S) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= N * N) return;
    const int i = idx / N, j = idx % N;
    const int a = min(i, j), b = max(i, j);
    double s = 0.0;
    int q = 0;
    for (; q + 8 <= nseg; q += 8) {                // eight loads in flight, added in order
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(q + u) * ldS * ldS + (size_t)a * ldS + b];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; q < nseg; ++q) s += part[(size_t)q * ldS * ldS + (size_t)a * ldS + b];
    S[idx] = s;
}

// Cyclic Jacobi on the symmetric N x N matrix S, one workgroup: each round
// applies N'/2 disjoint rotations (round-robin pairing, N' = N rounded up to
// even, the extra index is a dummy) to the rows and the columns.  Sweeps continue
// while the off-diagonal mass exceeds (1e-15)^2 of the diagonal mass, at most
// max_sweeps (every thread takes the same decision).  On exit diag(S) holds the
// eigenvalues (and S the rotated matrix, for a further pass); the rotations of
// every round (c, s, NaN-free) are left in rot [sweep (N' - 1) + round][N'/2][2]
// for k_jacobi_vectors.  sweeps_out[1] = the sweeps of this pass, sweeps_out[0]
// those of all (`more`: this pass continues an earlier one).
// Bound by the latency of its rounds (N=128: 127 a sweep, each a pass over the
// matrix between barriers), so the matrix stays in LDS where it fits (LDS =
// true: N <= kJacobiLdsN, 8 N^2 bytes), a pass rotates rows and columns of a
// 2 x 2 block together, and the eigenvectors, whose rows are independent of
// each other, are left to a kernel that uses the whole chip.  N=128: 58.0 ms
// with S and U in global memory and separate row and column passes, 6.5 ms with
// them in LDS, 3.4 ms and 0.4 for the vectors as it is.
constexpr int kJacobiThreads = 1024;
constexpr int kJacobiLdsN = 140;
template <bool LDS>
__global__ __launch_bounds__(kJacobiThreads) void k_jacobi(double* __restrict__ S, int N, int max_sweeps,
                                                           int more, double* __restrict__ rot,
                                                           int* __restrict__ sweeps_out) {
    extern __shared__ double lds[];
    __shared__ double cs[128][2];
    __shared__ int pq[128][2];
    __shared__ double red[kJacobiThreads / 64][2];
    __shared__ int stop;
    const int Np = N + (N & 1);
    const int half = Np / 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kWaves = kJacobiThreads / 64;
    double* A = LDS ? lds : S;
    if constexpr (LDS) {
        for (int idx = tid; idx < N * N; idx += kJacobiThreads) A[idx] = S[idx];
        __syncthreads();
    }
    int sweep = 0;
    for (; sweep < max_sweeps; ++sweep) {
        // convergence test on the current matrix
        double off = 0.0, dia = 0.0;
        for (int i = wave; i < N; i += kWaves)
            for (int j = lane; j < N; j += 64) {
                const double v = A[i * N + j];
                if (i == j) dia += v * v; else off += v * v;
            }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            off += __shfl_xor(off, m);
            dia += __shfl_xor(dia, m);
        }
        if (lane == 0) { red[wave][0] = off; red[wave][1] = dia; }
        __syncthreads();
        if (tid == 0) {
            double o = 0.0, d = 0.0;
            for (int k = 0; k < kWaves; ++k) { o += red[k][0]; d += red[k][1]; }
            stop = !(o > 1e-30 * d);
        }
        __syncthreads();
        if (stop) break;
        for (int round = 0; round < Np - 1; ++round) {
            // pairing: index 0 fixed, the others rotate
            if (tid < half) {
                auto player = [&](int slot) { return slot == 0 ? 0 : 1 + (slot - 1 + round) % (Np - 1); };
                const int p = player(tid), q = player(Np - 1 - tid);
                const int a = min(p, q), b = max(p, q);
                double c = 1.0, s = 0.0;
                if (b < N) {
                    const double apq = A[a * N + b];
                    if (apq != 0.0) {
                        const double app = A[a * N + a], aqq = A[b * N + b];
                        const double tau = (aqq - app) / (2.0 * apq);
                        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                        c = 1.0 / sqrt(1.0 + t * t);
                        s = t * c;
                    }
                }
                cs[tid][0] = c; cs[tid][1] = s;
                pq[tid][0] = a; pq[tid][1] = b;
                double* out = rot + (((size_t)sweep * (Np - 1) + round) * half + tid) * 2;
                out[0] = c;
                out[1] = s;
            }
            __syncthreads();
            // S <- J^T S J, one 2 x 2 block (rows of pair r1, columns of pair r2)
            // at a time: r1 uniform over a wave, r2 over its lanes
            for (int r2 = lane; r2 < half; r2 += 64) {
                const int a2 = pq[r2][0], b2 = pq[r2][1];
                const double c2 = cs[r2][0], s2 = cs[r2][1];
                const bool two = b2 < N;
                for (int r1 = wave; r1 < half; r1 += kWaves) {
                    const int a1 = pq[r1][0], b1 = pq[r1][1];
                    const double c1 = cs[r1][0], s1 = cs[r1][1];
                    double* ra = A + a1 * N;
                    double xa = ra[a2], ya = two ? ra[b2] : 0.0;
                    if (b1 < N) {
                        double* rb = A + b1 * N;
                        const double xb = rb[a2], yb = two ? rb[b2] : 0.0;
                        const double ub = s1 * xa + c1 * xb, vb = s1 * ya + c1 * yb;
                        xa = c1 * xa - s1 * xb;
                        ya = c1 * ya - s1 * yb;
                        rb[a2] = two ? c2 * ub - s2 * vb : ub;
                        if (two) rb[b2] = s2 * ub + c2 * vb;
                    }
                    ra[a2] = two ? c2 * xa - s2 * ya : xa;
                    if (two) ra[b2] = s2 * xa + c2 * ya;
                }
            }
            __syncthreads();
        }
    }
    if constexpr (LDS)
        for (int idx = tid; idx < N * N; idx += kJacobiThreads) S[idx] = A[idx];
    if (tid == 0) {
        sweeps_out[1] = sweep;
        sweeps_out[0] = (more ? sweeps_out[0] : 0) + sweep;
    }
}

// U <- I J_1 J_2 ... : the rotations of a pass of k_jacobi applied to the rows of
// the identity, or with `more` of U, one wave per row (rows do not meet), the row in LDS and the
// rotations of a round read one lane per pair.  The columns of U are the
// eigenvectors.
__global__ __launch_bounds__(64) void k_jacobi_vectors(const double* __restrict__ rot, const int* __restrict__ sweeps,
                                                       int N, int more, double* __restrict__ U) {
    __shared__ double row[256];
    const int Np = N + (N & 1), half = Np / 2;
    const int k = blockIdx.x, lane = threadIdx.x;
    const int rounds = sweeps[1] * (Np - 1);
    if (more && rounds == 0) return;
    for (int j = lane; j < N; j += 64) row[j] = more ? U[(size_t)k * N + j] : j == k ? 1.0 : 0.0;
    __syncthreads();
    const double2* rt = (const double2*)rot;
    constexpr int kAhead = 4;                        // rounds of rotations in flight
    double2 next[kAhead][2];
    auto load = [&](int rd, double2 (&v)[2]) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            v[u] = rt[(size_t)min(rd, max(rounds - 1, 0)) * half + min(lane + 64 * u, half - 1)];
    };
    if (rounds > 0)
#pragma unroll
        for (int u = 0; u < kAhead; ++u) load(u, next[u]);
    for (int rd0 = 0; rd0 < rounds; rd0 += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int rd = rd0 + u;
            double2 v[2] = {next[u][0], next[u][1]};
            load(rd + kAhead, next[u]);
            if (rd < rounds) {
                const int round = rd % (Np - 1);
                auto player = [&](int slot) { return slot == 0 ? 0 : 1 + (slot - 1 + round) % (Np - 1); };
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const int r = lane + 64 * w;
                    if (r < half) {
                        const int p = player(r), q = player(Np - 1 - r);
                        const int a = min(p, q), b = max(p, q);
                        if (b < N) {
                            const double c = v[w].x, s = v[w].y;
                            const double ua = row[a], ub = row[b];
                            row[a] = c * ua - s * ub;
                            row[b] = s * ua + c * ub;
                        }
                    }
                }
            }
            __syncthreads();                         // one wave: orders the rounds' LDS accesses
        }
    }
    for (int j = lane; j < N; j += 64) U[(size_t)k * N + j] = row[j];
}

// X = U diag(lambda^-1/2) U^T with lambda = diag(S) after the Jacobi sweeps.
__global__ void k_inv_sqrt(const double* __restrict__ S, const double* __restrict__ U, int N, double* __restrict__ X) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= N * N) return;
    const int i = idx / N, j = idx % N;
    const int a = min(i, j), b = max(i, j);       // exact symmetry of X
    double s = 0.0;
    for (int k = 0; k < N; ++k) s += U[(size_t)a * N + k] * U[(size_t)b * N + k] / sqrt(S[(size_t)k * N + k]);
    X[idx] = s;
}

// phi[i][g] = sum_j X[i][j] chi[j][g] on FP64 MFMA.  Workgroup: 64 rows of X in
// LDS (transposed, [j][64], zero past N), four waves of 64 points each; the
// next four rows of chi are in flight while four are multiplied.  N=128,
// 150 000 points: 2620 us with one thread per output.
constexpr int kApplyPoints = 256;
__global__ __launch_bounds__(256, 2) void k_apply_X(const double* __restrict__ X, const double* __restrict__ chi, int N,
                                                    int Ng, double* __restrict__ phi) {
    extern __shared__ double xs[];                 // [N rounded up to 4][64]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, kq = lane >> 4;
    const int i0 = blockIdx.y * 64;
    const int N4 = (N + 3) / 4 * 4;
    for (int idx = threadIdx.x; idx < N4 * 64; idx += 256) {
        const int j = idx >> 6, i = i0 + (idx & 63);
        xs[idx] = i < N && j < N ? X[(size_t)j * N + i] : 0.0;      // X is symmetric
    }
    __syncthreads();
    const int g0 = blockIdx.x * kApplyPoints + wave * 64;
    if (g0 >= Ng) return;
    d4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = (d4){0.0, 0.0, 0.0, 0.0};
    int col[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) col[c] = min(g0 + 16 * c + l16, Ng - 1);
    double next[4];
    auto load = [&](int j) {
        const double* row = chi + (size_t)min(j + kq, N - 1) * Ng;
#pragma unroll
        for (int c = 0; c < 4; ++c) next[c] = row[col[c]];
    };
    load(0);
    for (int j = 0; j < N4; j += 4) {
        double b[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) b[c] = next[c];
        load(j + 4);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const double x = xs[(j + kq) * 64 + 16 * a + l16];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b[c], acc[a][c], 0, 0, 0);
        }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + 16 * a + kq + 4 * v;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int g = g0 + 16 * c + l16;
                if (i < N && g < Ng) phi[(size_t)i * Ng + g] = acc[a][c][v];
            }
        }
}

// Convergence record of the Jacobi solve: out[0] = sweeps taken, out[1] = the
// smallest eigenvalue (NaN if any is NaN).
__global__ void k_lowdin_status(const double* __restrict__ S, int N, const int* __restrict__ sweeps,
                                double* __restrict__ out) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double m = S[0];
    for (int i = 1; i < N; ++i) {
        const double v = S[(size_t)i * N + i];
        m = (v < m || v != v) ? v : m;
    }
    out[0] = (double)*sweeps;
    out[1] = m;
}

__global__ void k_diag_copy(const double* __restrict__ S, int N, double* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) out[i] = S[(size_t)i * N + i];
}

}  // namespace xtc
