// Closed-shell intermediates, two-body assembly and one-body reduction (FP64).
//
// Notation (Appendix B, eq. tcmf:inter), per grid point g, k and l over the
// occupied orbitals, x over the Cartesian components:
//   rho_rs = w phi_r phi_s      K_rs = V_r^s (3-vector)
//   W  = 2 sum_k K_kk           Wt = 2 sum_k rho_kk
//   Zt_rs = sum_k K_rk . K_ks   Z_rs = sum_k (rho_rk K_ks + K_rk rho_ks)
//   A_rs = W . K_rs - Zt_rs     B_rs = Wt/2 K_rs - Z_rs
// C = [rho; Kx; Ky; Kz] and D = [A; Bx; By; Bz] are [4][rows][ldP] arrays,
// and eq. tcmf:2el becomes M[P][R] = sum_g sum_c C_c[g][P] D_c[g][R].
#pragma once
#include "xtc_device.h"

namespace xtc {

// The orbitals of the reference density with the occupations of one spin
// channel, w[i] (gamma^s = sum_i w[i] |k[i]><k[i]|), and of both spins
// together, wt[i] (closed shell: wt = 2 w).  128 entries cover every problem
// the on-chip staging of the intermediates admits (nocc * N <= 5120).
constexpr int kMaxOcc = 128;
struct OccList {
    int32_t n;
    int32_t k[kMaxOcc];
    double w[kMaxOcc];
    double wt[kMaxOcc];
};

// --------------------------------------------------------------------------
// Intermediates.  One workgroup handles one grid point at a time (grid-stride
// over the rows of the chunk).  The occupied columns (rho_rk, K_rk) of that
// point are gathered into LDS as [nocc][N] of (rho, Kx, Ky, Kz) (each thread's loads of up to
// kIGather entries issued together); each thread then owns kITile x kITile
// output blocks (r-block <= s-block) of the upper triangle and accumulates
// Zt and Z over k with register blocking.  The kernel waits on its loads and
// barriers, so what matters is how many workgroups a CU holds and that K is
// loaded before the sums: 2 x 2 blocks (149 registers; 4 x 4 took 254 and had
// none left for K), in workgroups of as many waves as the blocks fill.  N=128,
// 7500 rows: 1572 -> 1075 us (8 reads and writes of 62.5 M pair values: 4.0 GB);
// N=160, 5000 rows: 2068 -> 1690; N=64, 20 000 rows: 1084 -> 575; N=8, 2000
// rows: 33 -> 12 us.  (16 bytes of LDS padding after every four entries, which
// 4 x 4 blocks needed, make no difference to 2 x 2 ones: N=128 1009 and 1005 us,
// N=64 583 and 576.)
// One spin channel s per launch: Z~ and Z carry the occupations n_k of that
// spin, W and W~ those of the total density.  Per-point scalars
// S[g] = (W~/2, W/2 (3), sum_k n_k A_kk, sum_k n_k B_kk (3)) feed the one-body
// reduction.
constexpr int kIGather = 4, kITile = 2;
__global__ __launch_bounds__(256) void k_intermediates(const double* __restrict__ rho_rows,
                                                       const double* __restrict__ K, int rows,
                                                       int ldP, int N, OccList occ,
                                                       double* __restrict__ D, size_t dstride,
                                                       double* __restrict__ S) {
    extern __shared__ d4 lcol[];                   // [nocc][N] of (rho, Kx, Ky, Kz)
    __shared__ double sW[4];                       // Wx, Wy, Wz, Wt
    const int n = occ.n;
    const size_t kstride = (size_t)rows * ldP;
    const int nb = (N + kITile - 1) / kITile;
    const int ntiles = nb * (nb + 1) / 2;
    const int nt = blockDim.x;
    for (int g = blockIdx.x; g < rows; g += gridDim.x) {
        const double* rg = rho_rows + (size_t)g * ldP;
        const double* kg = K + (size_t)g * ldP;
        // every thread issues the loads of up to kIGather entries before storing
        for (int base = threadIdx.x; base < n * N; base += kIGather * nt) {
            d4 e[kIGather];
#pragma unroll
            for (int u = 0; u < kIGather; ++u) {
                const int idx = base + nt * u;
                if (idx < n * N) {
                    const int kk = idx / N, r = idx % N;
                    const int P = pair_sym(r, occ.k[kk], N);
                    e[u] = (d4){rg[P], kg[P], kg[kstride + P], kg[2 * kstride + P]};
                }
            }
#pragma unroll
            for (int u = 0; u < kIGather; ++u)
                if (base + nt * u < n * N) lcol[base + nt * u] = e[u];
        }
        __syncthreads();
        if (threadIdx.x < 64) {
            // wave 0: W, Wt and the per-point scalars of the one-body reduction,
            // lanes over occupied k, then a fixed-pattern butterfly sum.
            const int lane = threadIdx.x;
            // W = sum_k wt_k K_kk and W~ = sum_k wt_k rho_kk over the total
            // density (Appendix A; 2 gamma for the closed shell, Appendix B);
            // w0..w2 = W/2, wt = W~/2
            double w0 = 0, w1 = 0, w2 = 0, wt = 0;
            for (int kk = 0; kk < n; ++kk) {           // every lane, same order
                const d4 e = lcol[kk * N + occ.k[kk]];
                const double nk = occ.wt[kk];
                wt = fma(nk, e.x, wt); w0 = fma(nk, e.y, w0); w1 = fma(nk, e.z, w1); w2 = fma(nk, e.w, w2);
            }
            wt *= 0.5; w0 *= 0.5; w1 *= 0.5; w2 *= 0.5;
            double a = 0, b0 = 0, b1 = 0, b2 = 0;
            for (int kk = lane; kk < n; kk += 64) {
                const int k = occ.k[kk];
                const d4 e = lcol[kk * N + k];       // (rho_kk, K_kk)
                double zt = 0, z0 = 0, z1 = 0, z2 = 0;
                for (int ll = 0; ll < n; ++ll) {
                    const d4 f = lcol[ll * N + k];   // (rho_kl, K_kl)
                    const double nl = occ.w[ll];
                    zt = fma(nl, f.y * f.y + f.z * f.z + f.w * f.w, zt);
                    z0 = fma(nl, 2.0 * f.x * f.y, z0); z1 = fma(nl, 2.0 * f.x * f.z, z1);
                    z2 = fma(nl, 2.0 * f.x * f.w, z2);
                }
                const double nk = occ.w[kk];
                a = fma(nk, 2.0 * (w0 * e.y + w1 * e.z + w2 * e.w) - zt, a);   // n_k A_kk
                b0 = fma(nk, wt * e.y - z0, b0); b1 = fma(nk, wt * e.z - z1, b1);
                b2 = fma(nk, wt * e.w - z2, b2);                               // n_k B_kk
            }
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
                a += __shfl_xor(a, m); b0 += __shfl_xor(b0, m);
                b1 += __shfl_xor(b1, m); b2 += __shfl_xor(b2, m);
            }
            if (lane == 0) {
                sW[0] = 2.0 * w0; sW[1] = 2.0 * w1; sW[2] = 2.0 * w2; sW[3] = 2.0 * wt;
                double* s = S + (size_t)g * 8;
                s[0] = wt; s[1] = w0; s[2] = w1; s[3] = w2;
                s[4] = a; s[5] = b0; s[6] = b1; s[7] = b2;
            }
        }
        __syncthreads();
        const double W0 = sW[0], W1 = sW[1], W2 = sW[2], hWt = 0.5 * sW[3];
        for (int t = threadIdx.x; t < ntiles; t += nt) {
            int bi, bj;
            pair_split(t, nb, bi, bj);
            double zt[kITile][kITile], z0[kITile][kITile], z1[kITile][kITile], z2[kITile][kITile];
#pragma unroll
            for (int i = 0; i < kITile; ++i)
#pragma unroll
                for (int j = 0; j < kITile; ++j) zt[i][j] = z0[i][j] = z1[i][j] = z2[i][j] = 0.0;
            int ri[kITile], sj[kITile];
#pragma unroll
            for (int i = 0; i < kITile; ++i) {
                ri[i] = min(kITile * bi + i, N - 1);
                sj[i] = min(kITile * bj + i, N - 1);
            }
            double kv[kITile][kITile][3];                      // K of the block
#pragma unroll
            for (int i = 0; i < kITile; ++i)
#pragma unroll
                for (int j = 0; j < kITile; ++j) {
                    const int P = pair_sym(ri[i], sj[j], N);
                    kv[i][j][0] = kg[P];
                    kv[i][j][1] = kg[kstride + P];
                    kv[i][j][2] = kg[2 * kstride + P];
                }
            for (int kk = 0; kk < n; ++kk) {
                const int row = kk * N;
                const double nk = occ.w[kk];
                d4 a[kITile], b[kITile];
#pragma unroll
                for (int i = 0; i < kITile; ++i) {
                    a[i] = lcol[row + ri[i]];
                    b[i] = nk * lcol[row + sj[i]];
                }
#pragma unroll
                for (int i = 0; i < kITile; ++i)
#pragma unroll
                    for (int j = 0; j < kITile; ++j) {
                        zt[i][j] = fma(a[i].y, b[j].y, fma(a[i].z, b[j].z, fma(a[i].w, b[j].w, zt[i][j])));
                        z0[i][j] = fma(a[i].x, b[j].y, fma(a[i].y, b[j].x, z0[i][j]));
                        z1[i][j] = fma(a[i].x, b[j].z, fma(a[i].z, b[j].x, z1[i][j]));
                        z2[i][j] = fma(a[i].x, b[j].w, fma(a[i].w, b[j].x, z2[i][j]));
                    }
            }
#pragma unroll
            for (int i = 0; i < kITile; ++i)
#pragma unroll
                for (int j = 0; j < kITile; ++j) {
                    const int r = kITile * bi + i, s = kITile * bj + j;
                    if (r < N && s < N && r <= s) {
                        const int P = pair_index(r, s, N);
                        const double k0 = kv[i][j][0], k1 = kv[i][j][1], k2 = kv[i][j][2];
                        double* dg = D + (size_t)g * ldP + P;
                        dg[0] = fma(W0, k0, fma(W1, k1, W2 * k2)) - zt[i][j];
                        dg[dstride] = hWt * k0 - z0[i][j];
                        dg[2 * dstride] = hWt * k1 - z1[i][j];
                        dg[3 * dstride] = hWt * k2 - z2[i][j];
                    }
                }
        }
        // padding columns (the adjoint sums over whole 16-column blocks of D)
        for (int P = N * (N + 1) / 2 + threadIdx.x; P < ldP; P += nt) {
            double* dg = D + (size_t)g * ldP + P;
            dg[0] = dg[dstride] = dg[2 * dstride] = dg[3 * dstride] = 0.0;
        }
        __syncthreads();
    }
}

// --------------------------------------------------------------------------
// V2[p][q][r][s] = -(M2[P][R] + M1[R][P]).  Closed shell: M1 = M2 = M, and all
// eight index symmetries hold bitwise because the sum does not depend on the
// order of its terms.  Open shell, spins (s, t) of (pq, rs): M2 = M^t, M1 = M^s
// (Appendix A, [Delta U]^{st}[pq, rs] = -(f^t(pq, rs) + f^s(rs, pq))).
// Bound by the write of V2 (2.1 GB at N=128).  Two steps over slabs of rows P:
// the packed sums W[P - P0][R] in 32 x 32 tiles, the transposed term through
// LDS, and then row P of W written to (p, q) and (q, p).  N=128: 4.01 ms with
// every element reading M[R][P] down a column, 0.35 + 0.85 ms now.
__global__ __launch_bounds__(256) void k_sym_sum(const double* __restrict__ M1, const double* __restrict__ M2, int ldP,
                                                 int P0, double* __restrict__ W) {
    __shared__ double t[32][33];
    const int Rt = blockIdx.x * 32, Pt = P0 + blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int i = 0; i < 32; i += 8) t[ty + i][tx] = M1[(size_t)(Rt + ty + i) * ldP + Pt + tx];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; i += 8)
        W[(size_t)(Pt - P0 + ty + i) * ldP + Rt + tx] = -(M2[(size_t)(Pt + ty + i) * ldP + Rt + tx] + t[tx][ty + i]);
}

// One workgroup: rows r of a tile of kExpandRows, all s, of one P.  The values
// with s >= r are read along s; those with s < r, whose packed index runs along
// r, come 16 consecutive r at a time through LDS.
constexpr int kExpandRows = 16;
__global__ __launch_bounds__(256) void k_expand_V2(const double* __restrict__ W, int ldP, int P0, int N,
                                                   double* __restrict__ V2) {
    __shared__ double t[kExpandRows][257];
    const int P = P0 + blockIdx.y, r0 = blockIdx.x * kExpandRows;
    int p, q;
    pair_split(P, N, p, q);
    const double* row = W + (size_t)blockIdx.y * ldP;
    const int rj = threadIdx.x & (kExpandRows - 1);
    for (int s = threadIdx.x / kExpandRows; s < min(N, r0 + kExpandRows); s += 256 / kExpandRows) {
        const int r = r0 + rj;
        if (r < N && s < r) t[rj][s] = row[pair_index(s, r, N)];
    }
    __syncthreads();
    const size_t NN = (size_t)N * N;
    double* pq = V2 + ((size_t)p * N + q) * NN;
    double* qp = V2 + ((size_t)q * N + p) * NN;
    const int rows = min(kExpandRows, N - r0);
    int r = 0, s = threadIdx.x;
    while (s >= N) {
        s -= N;
        ++r;
    }
    while (r < rows) {
        const double v = s < r0 + r ? t[r][s] : row[pair_index(r0 + r, s, N)];
        const size_t o = (size_t)(r0 + r) * N + s;
        pq[o] = v;
        if (p != q) qp[o] = v;
        s += 256;
        while (s >= N) {
            s -= N;
            ++r;
        }
    }
}

// --------------------------------------------------------------------------
// One-body reduction, term 1 (diagonal-sum terms), partial over grid splits:
//   T1[split][P] = sum_{g in split} rho_P a + K_P.b + rb A_P + kb.B_P
// with rb = W~/2, kb = W/2 and (a, b) = sum_k n_k (A_kk, B_kk) of this channel,
// or, when S2 (the other spin channel) is given, the mean over both channels
// (Appendix A: the sum over the spin tau of [Delta U]^{s tau} gamma^tau).
__global__ __launch_bounds__(256) void k_onebody_T1(const double* __restrict__ rho_rows,
                                                    const double* __restrict__ K,
                                                    const double* __restrict__ D, size_t dstride,
                                                    const double* __restrict__ S, const double* __restrict__ S2,
                                                    int rows, int ldP, int Npair, double* __restrict__ T1) {
    const int P = blockIdx.x * blockDim.x + threadIdx.x;
    const int split = blockIdx.y, nsplit = gridDim.y;
    if (P >= Npair) return;
    const size_t kstride = (size_t)rows * ldP;
    const int gb = (int)(((long)rows * split) / nsplit), ge = (int)(((long)rows * (split + 1)) / nsplit);
    double acc = 0.0;
    for (int g = gb; g < ge; ++g) {
        const double* s = S + (size_t)g * 8;
        double ab[4] = {s[4], s[5], s[6], s[7]};
        if (S2) {
            const double* s2 = S2 + (size_t)g * 8;
#pragma unroll
            for (int i = 0; i < 4; ++i) ab[i] = 0.5 * (ab[i] + s2[4 + i]);
        }
        const size_t o = (size_t)g * ldP + P;
        acc = fma(rho_rows[o], ab[0], acc);
        acc = fma(K[o], ab[1], fma(K[kstride + o], ab[2], fma(K[2 * kstride + o], ab[3], acc)));
        acc = fma(D[o], s[0], acc);
        acc = fma(D[dstride + o], s[1], fma(D[2 * dstride + o], s[2], fma(D[3 * dstride + o], s[3], acc)));
    }
    T1[(size_t)split * ldP + P] = acc;
}

// One-body reduction, exchange term, partial over grid splits:
//   E[split][p][q] = sum_{g in split} sum_k n_k sum_c C_c[g][pair(p,k)] D_c[g][pair(k,q)]
// on FP64 MFMA, the sum over k in groups of 4 as the MFMA's inner index and
// the sums over g and c in sequence.  Four waves share the rows of one tile of
// 16 TB x 16 TB outputs (wave w takes g = w, w + 4, ...) and meet in LDS in a
// fixed order.  For a fixed k the pairs (p, k) of 16 consecutive p are (almost
// always) 16 consecutive columns, so each lane loads its operand straight from
// the rows; the columns are found once per group of k, outside the loop over
// g.  The next component's operands are in flight while one is multiplied.
// N=128, 16 occupied, 7500 rows: 1000 -> 408 us; N=64, 20, 5000 rows: 621 -> 98;
// N=24, 6, 4001 rows: 148 -> 12.5; N=8, 2, 2000 rows: 37 -> 4.3 (a thread per
// 4 x 4 outputs over columns staged in LDS per point and component before).
template <int TB>
__global__ __launch_bounds__(256, 2) void k_onebody_E(const double* __restrict__ rho_rows,
                                                   const double* __restrict__ K,
                                                   const double* __restrict__ D, size_t dstride,
                                                   int rows, int ldP, int N, OccList occ,
                                                   double* __restrict__ E) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = occ.n;
    const int nt = (N + 16 * TB - 1) / (16 * TB);
    const int p0 = (blockIdx.x % nt) * 16 * TB, q0 = (blockIdx.x / nt) * 16 * TB;
    const int split = blockIdx.y, nsplit = gridDim.y;
    const int gb = (int)(((long)rows * split) / nsplit), ge = (int)(((long)rows * (split + 1)) / nsplit);
    const size_t kstride = (size_t)rows * ldP;
    const int l16 = lane & 15, kq = lane >> 4;
    d4 acc[TB][TB];
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = (d4){0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < n; k0 += 4) {
        const int kk = min(k0 + kq, n - 1), k = occ.k[kk];
        const bool on = k0 + kq < n;
        const double nk = occ.w[kk];
        int cp[TB], cq[TB];                            // this lane's columns (clamped past N)
#pragma unroll
        for (int i = 0; i < TB; ++i) {
            cp[i] = pair_sym(min(p0 + 16 * i + l16, N - 1), k, N);
            cq[i] = pair_sym(min(q0 + 16 * i + l16, N - 1), k, N);
        }
        double a[2][TB], b[2][TB];
        auto load = [&](int s, int g, int c) {
            const size_t o = (size_t)g * ldP;
            const double* C = c == 0 ? rho_rows + o : K + (size_t)(c - 1) * kstride + o;
            const double* Dg = D + (size_t)c * dstride + o;
#pragma unroll
            for (int i = 0; i < TB; ++i) {
                a[s][i] = C[cp[i]];
                b[s][i] = Dg[cq[i]];
            }
        };
        int g = gb + wave;
        if (g < ge) load(0, g, 0);
        for (; g < ge; g += 4) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double av[TB], bv[TB];
#pragma unroll
                for (int i = 0; i < TB; ++i) {
                    av[i] = on ? a[c & 1][i] : 0.0;
                    bv[i] = on ? nk * b[c & 1][i] : 0.0;
                }
                if (c < 3) load((c + 1) & 1, g, c + 1);
                else load(0, min(g + 4, ge - 1), 0);
#pragma unroll
                for (int i = 0; i < TB; ++i)
#pragma unroll
                    for (int j = 0; j < TB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    // waves 2, 3 onto 0, 1, then 1 onto 0
    __shared__ double red[2][4 * TB * TB][64];
#pragma unroll
    for (int step = 2; step >= 1; step >>= 1) {
        if (wave >= step && wave < 2 * step)
#pragma unroll
            for (int i = 0; i < TB; ++i)
#pragma unroll
                for (int j = 0; j < TB; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[wave - step][4 * (TB * i + j) + v][lane] = acc[i][j][v];
        __syncthreads();
        if (wave < step)
#pragma unroll
            for (int i = 0; i < TB; ++i)
#pragma unroll
                for (int j = 0; j < TB; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[i][j][v] += red[wave][4 * (TB * i + j) + v][lane];
        __syncthreads();
    }
    if (wave != 0) return;
    double* out = E + (size_t)split * N * N;
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = p0 + 16 * i + kq + 4 * v;    // logical row l/16 + 4v
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                const int q = q0 + 16 * j + l16;
                if (p < N && q < N) out[(size_t)p * N + q] = acc[i][j][v];
            }
        }
}

// Fold the split partials of one chunk into the packed FP64 accumulator:
//   h1acc[pair(p,q)] (+)= sum_s T1[s][P] - 1/2 (sum_s E[s][p][q] + sum_s E[s][q][p])
// 32 pairs per workgroup, the partials of each shared by kAccSlices threads
// (slice t takes s = t, t + kAccSlices, ...) whose sums meet in a fixed order:
// one thread per pair took 84-115 us of load latency, this takes 9 (N=8), 15
// (N=64) and 31 (N=128).
constexpr int kAccSlices = 8;
__global__ __launch_bounds__(256) void k_onebody_accumulate(const double* __restrict__ T1, int nsplit_t1,
                                                            const double* __restrict__ E, int nsplit_e, int ldP, int N,
                                                            double* __restrict__ h1acc, int accumulate) {
    __shared__ double red[kAccSlices][32];
    const int j = threadIdx.x & 31, slice = threadIdx.x >> 5;
    const int P = blockIdx.x * 32 + j;
    const int Npair = N * (N + 1) / 2;
    double v = 0.0;
    if (P < Npair) {
        int p, q;
        pair_split(P, N, p, q);
        double t = 0.0, e = 0.0;
#pragma unroll 4
        for (int s = slice; s < nsplit_t1; s += kAccSlices) t += T1[(size_t)s * ldP + P];
        const size_t NN = (size_t)N * N;
#pragma unroll 4
        for (int s = slice; s < nsplit_e; s += kAccSlices) e += E[s * NN + (size_t)p * N + q] + E[s * NN + (size_t)q * N + p];
        v = t - 0.5 * e;
    }
    red[slice][j] = v;
    __syncthreads();
    if (slice == 0 && P < Npair) {
#pragma unroll
        for (int s = 1; s < kAccSlices; ++s) v += red[s][j];
        h1acc[P] = accumulate ? h1acc[P] + v : v;
    }
}

// h1[p][q] = h1acc[pair(p,q)] (symmetric bitwise) for one spin channel, or for
// both (h1acc2, h1 + N^2) in the open-shell form.  E0 = -(2/3) sum_k n_k h1[k][k]
// (Appendix B), or -(1/3) sum_s sum_k n^s_k h1^s[k][k] (Appendix A), summed in
// occ order by one thread.
__global__ void k_onebody_finalize(const double* __restrict__ h1acc, const double* __restrict__ h1acc2, int N,
                                   OccList occ, OccList occ2, double* __restrict__ h1, double* __restrict__ E0) {
    const int pq = blockIdx.x * blockDim.x + threadIdx.x;
    if (pq < N * N) {
        const int p = pq / N, q = pq % N;
        h1[pq] = h1acc[pair_sym(p, q, N)];
        if (h1acc2) h1[N * N + pq] = h1acc2[pair_sym(p, q, N)];
    }
    if (pq == 0) {
        double e = 0.0;
        for (int kk = 0; kk < occ.n; ++kk) e = fma(occ.w[kk], h1acc[pair_index(occ.k[kk], occ.k[kk], N)], e);
        if (h1acc2) {
            for (int kk = 0; kk < occ2.n; ++kk)
                e = fma(occ2.w[kk], h1acc2[pair_index(occ2.k[kk], occ2.k[kk], N)], e);
            *E0 = -(1.0 / 3.0) * e;
        } else {
            *E0 = -(2.0 / 3.0) * e;
        }
    }
}

}  // namespace xtc
