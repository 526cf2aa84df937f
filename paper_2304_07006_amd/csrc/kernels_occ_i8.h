// Occupied-occupied block of K from exact integer products, for the
// reduced-precision forms:
//   K^x_P(g) = sum_g' d^x(g,g') rho_P(g')      (Theory, definition of V)
// over the occupied pairs P, to the accuracy of an FP64 evaluation, on the
// int8 matrix cores (v_mfma_i32_16x16x64_i8) instead of the FP64 ones.
//
// Both operands become fixed-point numbers of six balanced base-128 digits
// relative to a power-of-two scale: S_d bounds 2|d^x| for the Jastrow at
// hand (|d^x| <= |u'(r)|), and S_P is the power of two above twice the
// largest |rho_P(g')| of pair P.  With v = d / S_d (or rho / S_P) in
// [-1/2, 1/2]:
//   v = sum_{i=1..6} a_i 2^(-7 i) + e,   |e| <= 2^-43,
// a_1 and a_4 in [-64, 64], the others in [-64, 63] (digits centred on zero,
// so that rounding and dropped terms carry no sign bias).  The digit products
// a_i b_j with i + j <= 7 (21 of the 36) are summed exactly in int32, one
// accumulator per order i + j; each dropped product is at most 2^-44 S_d S_P
// and all of them together below 2.87e-13 S_d S_P.
// The orders are combined in FP64 per segment of at most kI8SegMax grid
// points (|an accumulator| <= 6 x 64 x 64 per point, < 2^31 over a segment),
// and the segments are summed in FP64 afterwards.
//
// Digit tiles are laid out as the MFMA consumes them: one 16-byte operand
// per lane, lane l standing for pair (or row) l % 16 and grid points
// 16 (l / 16) + e, e = 0..15, of a 64-point k-step (both operands use the
// same assignment, so the sum over the 64 points does not depend on the
// order the hardware gives the bytes).  The int32 result of lane l holds
// rows 4 (l / 16) + v, v = 0..3, of column l % 16.
#pragma once
#include "xtc_device.h"

namespace xtc {

typedef int i4 __attribute__((ext_vector_type(4)));

constexpr int kI8Digits = 6;          // digits per operand
constexpr int kI8Orders = 6;          // accumulated orders i + j = 2..7
constexpr int kI8Kb = 64;             // grid points per MFMA k-step
constexpr int kI8TileB = 64 * 16;     // bytes of one digit tile (64 lanes x 16 bytes)
constexpr int kI8SegMax = 65536;      // grid points per int32 segment
constexpr int kI8MaxCT = 9;           // 16-pair column tiles per wave
// Waves per workgroup of a kernel with CT column tiles: eight (two per SIMD)
// while their accumulators leave registers for that, else four.
constexpr int i8_waves(int ct) { return ct <= 5 ? 8 : 4; }

// The digit products a_i b_j kept (0-based, i + j <= 5), so ordered that
// consecutive products share their left operand and add to different orders.
constexpr int kI8Products = 21;
constexpr int kI8Left[kI8Products] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 2, 2, 2, 2, 3, 3, 3, 4, 4, 5};
constexpr int kI8Right[kI8Products] = {0, 1, 2, 3, 4, 5, 0, 1, 2, 3, 4, 0, 1, 2, 3, 0, 1, 2, 0, 1, 0};

// Power of two S > 2 m (1 for m = 0), so that |x| <= m gives |x| / S < 1/2.
__host__ __device__ inline double i8_scale(double m) {
    if (!(m > 0.0)) return 1.0;
    int e = 0;
    (void)frexp(m, &e);   // m < 2^e
    return ldexp(1.0, e + 1);
}

// The six digits of four values at once, from h = v 2^21 (|h| <= 2^20 plus
// rounding), packed four to a register (byte b of w[s]: digit s of value b):
// h = H + L 2^-21 + e with integers |H|, |L| <= 2^20 (+1) and |e| <= 2^-22,
// then each of H, L = t 2^14 + m 2^7 + l with m, l in [-64, 63] and
// t in [-64, 64].  The FP64 roundings go through the shifter 1.5 2^52 + 8256,
// whose low word is the rounded integer plus 8256 = 64 (2^7 + 1); that turns m
// and l into 64 more than themselves, in bits 7..13 and 0..6, which
// i8_fields takes out of four values together (38 integer instructions for
// the 24 digits of four values; one value at a time took 96).
__device__ __forceinline__ int i8_bytes(int a, int b, int sel) {
    return (int)__builtin_amdgcn_perm((unsigned)b, (unsigned)a, (unsigned)sel);
}
// bytes x in [0, 127] (bit 7 ignored) -> x - 64 as signed bytes
__device__ __forceinline__ int i8_center(int x) {
    const int y = (x & 0x7f7f7f7f) ^ 0x40404040;
    return y | ((y & 0x40404040) << 1);
}
__device__ __forceinline__ void i8_fields(const int (&u)[4], int& t, int& m, int& l) {
    const int w01 = i8_bytes(u[0], u[1], 0x05040100), w23 = i8_bytes(u[2], u[3], 0x05040100);   // low halves
    l = i8_center(i8_bytes(w01, w23, 0x06040200));
    m = i8_center(i8_bytes((int)((unsigned)w01 >> 7), (int)((unsigned)w23 >> 7), 0x06040200));
    const int t01 = i8_bytes(u[0] >> 14, u[1] >> 14, 0x0c0c0400), t23 = i8_bytes(u[2] >> 14, u[3] >> 14, 0x04000c0c);
    t = t01 | t23;
}
__device__ __forceinline__ void i8_digits4(const double (&h)[4], int (&w)[kI8Digits]) {
    const double kShift = 6755399441055744.0 + 8256.0;   // 1.5 * 2^52 + 64 (2^7 + 1)
    int uh[4], ul[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const double th = h[b] + kShift;
        const double hr = th - kShift;
        const double tl = fma(h[b] - hr, 2097152.0, kShift);
        uh[b] = (int)__builtin_bit_cast(unsigned long long, th);
        ul[b] = (int)__builtin_bit_cast(unsigned long long, tl);
    }
    i8_fields(uh, w[0], w[1], w[2]);
    i8_fields(ul, w[3], w[4], w[5]);
}

// Per-pair largest |rho_P(g')| of the gathered occupied pairs
// (rho_occ[g'][ldO]), as the bit pattern of a non-negative double (ordered like the value), max-combined into amax[P]
// (zero before the first launch).  Grid: (column tiles of 16 pairs, row
// chunks); 256 threads: 16 pairs x 16 rows at a time.
__global__ __launch_bounds__(256) void k_occ_absmax(const double* __restrict__ rho_occ, int ngp, int ldO, int nOP,
                                                    int rows_per_block, unsigned long long* __restrict__ amax) {
    __shared__ double red[256];
    const int j = threadIdx.x & 15, rs = threadIdx.x >> 4;
    const int P = blockIdx.x * 16 + j;
    const int r0 = blockIdx.y * rows_per_block, r1 = min(ngp, r0 + rows_per_block);
    double m = 0.0;
    if (P < nOP) {
        const double* col = rho_occ + P;
        for (int g = r0 + rs; g < r1; g += 16) m = fmax(m, fabs(col[(size_t)g * ldO]));
    }
    red[threadIdx.x] = m;
    __syncthreads();
    if (rs == 0 && P < nOP) {
        for (int i = 1; i < 16; ++i) m = fmax(m, red[16 * i + j]);
        atomicMax(amax + P, __builtin_bit_cast(unsigned long long, m));
    }
}

// Stage blocks of the main kernel, one per k-step kb and column group: the
// digit tiles of rho for the group's CT column tiles, [ct][s][lane] (16 bytes
// each; pairs >= nOP are zero).  In LDS the positions (x, y, z, 0) of the 64
// points of k-steps kb + 1 and kb + 2 (zero past the grid) stand behind them,
// and padding to whole 8 KB, one 1 KB chunk per wave and round (4 KB with four
// waves), so that the loads are the same straight line for every wave: with a
// branch for the position chunks a chunk of 7500 rows at N=128 took 141.1
// instead of 140.6 ms.
template <int CT> struct OccI8Stage {
    static constexpr int kDigitB = CT * kI8Digits * kI8TileB;
    static constexpr int kDigitChunks = kDigitB / 1024;                      // 1 KB direct-load chunks
    static constexpr int kRounds = (kDigitChunks + 2 * kI8Kb * 32 / 1024 + i8_waves(CT) - 1) / i8_waves(CT);
    static constexpr int kBlockB = 1024 * i8_waves(CT) * kRounds;            // in LDS
};

// Digits: one thread per (kb, column tile ct8 of nct8 = groups x CT, lane).
template <int CT>
__global__ __launch_bounds__(256) void k_occ_slice(const double* __restrict__ rho_occ, int ngp, int ldO, int nOP,
                                                   int groups, const unsigned long long* __restrict__ amax,
                                                   char* __restrict__ stages) {
    typedef OccI8Stage<CT> S;
    const int nct8 = groups * CT;
    const size_t n = (size_t)(ngp / kI8Kb) * nct8 * 64;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(idx & 63);
        const size_t rest = idx >> 6;
        const int ct8 = (int)(rest % nct8);
        const size_t kb = rest / nct8;
        const int P = ct8 * 16 + (lane & 15);
        const int gq = (int)kb * kI8Kb + 16 * (lane >> 4);
        const bool on = P < nOP;
        const double hs = on ? 2097152.0 / i8_scale(__builtin_bit_cast(double, amax[P])) : 0.0;
        const double* col = rho_occ + (on ? P : 0);
        int w[kI8Digits][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double h[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) h[b] = (on ? col[(size_t)(gq + 4 * k + b) * ldO] : 0.0) * hs;
            int d[kI8Digits];
            i8_digits4(h, d);
#pragma unroll
            for (int s = 0; s < kI8Digits; ++s) w[s][k] = d[s];
        }
        char* blk = stages + (kb * groups + ct8 / CT) * S::kDigitB + (size_t)(ct8 % CT) * kI8Digits * kI8TileB;
#pragma unroll
        for (int s = 0; s < kI8Digits; ++s)
            *(i4*)(blk + (s * 64 + lane) * 16) = (i4){w[s][0], w[s][1], w[s][2], w[s][3]};
    }
}

// Word 3 of a raw (untyped, unswizzled) buffer descriptor on gfx9-family GPUs.
constexpr int kI8RawBufferWord3 = 0x00020000;

// The block for rows [g0, g0 + rows).  Each wave owns one task: 16 rows
// (row block rb) and one component x of d, for the CT column tiles of column
// group blockIdx.z, so its accumulators are CT x 6 orders x 4 registers; task
// W blockIdx.x + wave is row block task / 3, component task % 3 (waves past
// the last task only help).  blockIdx.y is the segment of seg_kb k-steps.
// A pipeline of three stages, one barrier per k-step: while the MFMAs consume
// the digits of k-step t (21 CT of them), the wave makes the digits of its d^x
// for k-step t + 1 (16 values per lane) from S u'(r)/r, which the workgroup
// computed together into LDS one k-step before, each value once for its row
// block's components, and shares in computing that for k-step t + 2.  (Each
// component's wave computing its own u'/r, half of the VALU work that bounds the
// kernel, took 11.2 ms for 136 pairs, 7500 rows, 150 000 points and 4.2 ms for 78
// pairs, 5000 rows, 100 000 points, power Jastrow; now 10.2 and 3.4.)
// Each stage block (stages[kb][group], OccI8Stage) and the positions behind it
// are copied by direct 16-byte buffer-to-LDS loads one k-step ahead into the
// other of two statically named buffers.  part[seg][x][r][ldK] = the FP64 value of the segment's sum, for
// pair columns 16 (blockIdx.z CT + ct) + l % 16.
template <int KIND, int CT>
__global__ __launch_bounds__(64 * i8_waves(CT), 1) void k_build_K_occ_i8(
    const d4* __restrict__ pos, const char* __restrict__ stages, int groups, int ngp, int g0, int rows, int n_rb,
    JasDev J, double sd, const unsigned long long* __restrict__ amax, double* __restrict__ part, int ldK, int seg_kb) {
    typedef OccI8Stage<CT> S;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    constexpr int W = i8_waves(CT);
    constexpr int kSlots = W == 8 ? 4 : 2;               // row blocks that W consecutive tasks can touch
    constexpr int kPairs = kSlots * 512 / (64 * W);      // pairs of u'/r values per thread and k-step
    // u'/r of a k-step: [row block][point / 16][pair of points][row][2]
    typedef double FTile[kSlots][4][8][16][2];
    __shared__ __attribute__((aligned(1024))) char sm0[S::kBlockB];
    __shared__ __attribute__((aligned(1024))) char sm1[S::kBlockB];
    __shared__ __attribute__((aligned(1024))) char smp[2 * kI8Kb * 32];
    __shared__ __attribute__((aligned(16))) FTile sF0;
    __shared__ __attribute__((aligned(16))) FTile sF1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int task0 = W * blockIdx.x, task = task0 + wave;
    const int live = __builtin_amdgcn_readfirstlane(task < 3 * n_rb ? 1 : 0);
    const int rb0 = task0 / 3;
    const int nslots = min(task0 + W - 1, 3 * n_rb - 1) / 3 - rb0 + 1;
    const int rb = live ? task / 3 : rb0;
    const int comp = live ? task % 3 : 0;
    const int cg = blockIdx.z;
    const int nkb = ngp / kI8Kb;
    const int kb0 = blockIdx.y * seg_kb;
    const int nst = min(seg_kb, nkb - kb0);
    const int q = lane >> 4, l16 = lane & 15;
    const d4 pg = pos[g0 + min(rb * 16 + l16, rows - 1)];
    const double pc = comp == 0 ? pg.x : comp == 1 ? pg.y : pg.z;
    const double hs = 2097152.0 / sd;   // digits of d / sd from d 2^21 / sd
    const uint32_t loff = 16 * lane;

    // stage t: the block of k-step kb0 + t
    auto issue = [&](int t, char* buf) {
        const int kb = kb0 + t;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(stages + ((size_t)kb * groups + cg) * S::kDigitB), (short)0, S::kDigitB, kI8RawBufferWord3);
        // positions past the grid's last point read as zero
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(pos + (size_t)(kb + 1) * kI8Kb), (short)0, 32 * min(2 * kI8Kb, ngp - (kb + 1) * kI8Kb),
            kI8RawBufferWord3);
#pragma unroll
        for (int i = 0; i < S::kRounds; ++i) {
            const int off = 1024 * (wave + W * i);
            // (chunks past the positions read as zero)
            const bool digits = W * (i + 1) <= S::kDigitChunks || off < S::kDigitB;
            const int src = digits ? off : off - S::kDigitB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(digits ? rs : rp, (lds_ptr)(buf + off), 16, loff, src, 0, 0);
        }
    };

    // u'/r role: pair i of this thread is row block i * W / 8 .., points 16 fq +
    // 2 fe, + 1, row threadIdx % 16
    double rx[kSlots], ry[kSlots], rz[kSlots];
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        const d4 p = pos[g0 + min((rb0 + s) * 16 + l16, rows - 1)];
        rx[s] = p.x;
        ry[s] = p.y;
        rz[s] = p.z;
    }
    auto share = [&](int i, const char* p64, FTile& F) {
        const int idx = threadIdx.x + 64 * W * i;
        const int slot = (64 * W * i) / 512;             // uniform: 512 pairs per row block
        const int fe = (idx >> 4) & 7, fq = (idx >> 7) & 3;
        const double* c = (const double*)(p64 + 32 * (16 * fq + 2 * fe));
        double* o = F[slot][fq][fe][l16];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const double dx = rx[slot] - c[4 * b], dy = ry[slot] - c[4 * b + 1], dz = rz[slot] - c[4 * b + 2];
            const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, kR2FloorF64)));
            o[b] = du_over_r_nz_f64<KIND>(r2, J, hs);
        }
    };
    auto share_all = [&](const char* p64, FTile& F) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i)
            if ((64 * W * i) / 512 < nslots) share(i, p64, F);
    };
    // digits of d^comp for this lane's row and points 16 q + 4 k + b, b = 0..3,
    // of the k-step whose positions are at p64 and u'/r in F
    auto digits4 = [&](const char* p64, const FTile& F, int k, i4 (&A)[kI8Digits]) {
        double h[4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
            h[b] = (pc - ((const double*)(p64 + 32 * (16 * q + 4 * k + b)))[comp]) *
                   F[rb - rb0][q][2 * k + b / 2][l16][b % 2];
        int d[kI8Digits];
        i8_digits4(h, d);
#pragma unroll
        for (int s = 0; s < kI8Digits; ++s) A[s][k] = d[s];
    };

    i4 acc[CT][kI8Orders];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int o = 0; o < kI8Orders; ++o) acc[c][o] = (i4){0, 0, 0, 0};
    i4 A[kI8Digits];

    // one k-step from `buf`, then the wait for this wave's loads of the next
    // stage and the barrier that publishes everyone's (and ends all reads of
    // this one).  With two waves per SIMD one wave's MFMAs cover the other's
    // generation.  With one (CT > 5), left to itself the compiler issues the
    // two one after the other: the k-step then runs in four fenced quarters,
    // each with a quarter of the MFMAs and the VALU work, issued as one MFMA
    // and its share of that work in turn.
    auto stage = [&](const char* buf, const FTile& R, FTile& F) {
        const char* pos1 = buf + S::kDigitB;             // positions of k-step t + 1
        const char* pos2 = pos1 + 32 * kI8Kb;            // and t + 2
        auto read_b = [&](int c, i4 (&b)[kI8Digits]) {
#pragma unroll
            for (int s = 0; s < kI8Digits; ++s)
                b[s] = *(const i4*)(buf + ((c * kI8Digits + s) * 64 + lane) * 16);
        };
        if (!live || CT <= 5) share_all(pos2, F);
        if (live) {
            i4 An[kI8Digits];
            if constexpr (CT <= 5) {
#pragma unroll
                for (int k = 0; k < 4; ++k) digits4(pos1, R, k, An);
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    i4 b[kI8Digits];
                    read_b(c, b);
#pragma unroll
                    for (int j = 0; j < kI8Products; ++j)
                        acc[c][kI8Left[j] + kI8Right[j]] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                            A[kI8Left[j]], b[kI8Right[j]], acc[c][kI8Left[j] + kI8Right[j]], 0, 0, 0);
                }
            } else {
                static_assert(CT <= 5 || kPairs == 4, "one pair of u'/r values per quarter");
                constexpr int kMfma = kI8Products * CT;
                constexpr int kValu = KIND == 0 ? 112 : 144;   // VALU instructions of a quarter
                constexpr int kPer = (4 * kValu + kMfma - 1) / kMfma;
                i4 b[2][kI8Digits];
                read_b(0, b[0]);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    __builtin_amdgcn_sched_barrier(0);
                    digits4(pos1, R, k, An);
                    share(k, pos2, F);
#pragma unroll
                    for (int m = kMfma * k / 4; m < kMfma * (k + 1) / 4; ++m) {
                        const int c = m / kI8Products, j = m % kI8Products;
                        if (j == 0 && c + 1 < CT) read_b(c + 1, b[(c + 1) & 1]);
                        acc[c][kI8Left[j] + kI8Right[j]] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                            A[kI8Left[j]], b[c & 1][kI8Right[j]], acc[c][kI8Left[j] + kI8Right[j]], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, 10, 0);         // LDS reads
#pragma unroll
                    for (int m = kMfma * k / 4; m < kMfma * (k + 1) / 4; ++m) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // MFMA
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);      // LDS read
                        __builtin_amdgcn_sched_group_barrier(0x002, kPer, 0);   // VALU
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int s = 0; s < kI8Digits; ++s) A[s] = An[s];
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    };

    if (nst > 0) {
        // positions of the first two k-steps (zero past the grid), then the
        // first one's stage, u'/r of both and the digits of the first
        const int left = min(2 * kI8Kb, ngp - kb0 * kI8Kb);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(pos + (size_t)kb0 * kI8Kb), (short)0, left * 32, kI8RawBufferWord3);
        if (wave < 4)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rp, (lds_ptr)(smp + 1024 * wave), 16, loff, 1024 * wave, 0, 0);
        issue(0, sm0);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        share_all(smp, sF0);
        share_all(smp + 32 * kI8Kb, sF1);
        __syncthreads();
        if (live) {
#pragma unroll
            for (int k = 0; k < 4; ++k) digits4(smp, sF0, k, A);
        }
        __syncthreads();                                  // before stage 0 writes sF0
    }
    int t = 0;
    for (; t + 1 < nst; t += 2) {
        issue(t + 1, sm1);
        stage(sm0, sF1, sF0);
        if (t + 2 < nst) issue(t + 2, sm0);
        stage(sm1, sF0, sF1);
    }
    if (t < nst) stage(sm0, sF1, sF0);

    if (!live) return;
    double* out = part + (size_t)blockIdx.y * 3 * rows * ldK;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int P = 16 * (cg * CT + c) + (lane & 15);
        const double sc = sd * i8_scale(__builtin_bit_cast(double, amax[P]));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = rb * 16 + 4 * q + v;
            if (r < rows) {
                double s = 0.0;
#pragma unroll
                for (int o = kI8Orders - 1; o >= 0; --o) s += (double)acc[c][o][v] * ldexp(1.0, -7 * (o + 2));
                out[((size_t)comp * rows + r) * ldK + P] = s * sc;
            }
        }
    }
}

}  // namespace xtc
