// Launcher of the FP64 K build (build_f64.h).
#include "build_f64.h"

#include <algorithm>

#include "kernels_build_f64.h"

namespace xtc {

namespace {

constexpr int kCus = 256;   // compute units of an MI355X (launch shapes only)

// Most 16-column blocks per wave.  With eight, as with seven, one workgroup has a
// CU to itself (at N=128 112 x 2 columns reach 60.8 TFLOP/s, 64 x 2 66.2), and
// the cost below never takes eight.
constexpr int kMaxBlocks = 7;

// Workgroups of a shape that share a CU (24 nb accumulation registers and about
// 110 others, of 512 per lane).
int resident(int nb) { return nb >= 7 ? 1 : nb >= 3 ? 2 : 3; }

// Cycles of a SIMD per k-step of a wave: 64 per MFMA, 8 per VALU instruction
// that the MFMAs cannot hide (about 36 generate a d^x, shared by cw waves, and
// a few move operands), and an eighth more where no second wave covers the
// waits (N=128, 4000 rows against 20 000 points: 16 nb x cw columns of 96 x 2
// 70.1 TFLOP/s, 80 x 4 68.0, 64 x 2 66.2, 112 x 2 alone on its SIMD 60.8).
double step_cycles(int nb, int cw) {
    return (192.0 * nb + 8.0 * (36.0 / cw + 4.0)) * (resident(nb) == 1 ? 1.125 : 1.0);
}

}  // namespace

KF64Plan kf64_columns(int cols, int ld) {
    KF64Plan best{1, 2, 0, 1, 0};
    double best_cost = 1e300;
    for (int nb = 1; nb <= kMaxBlocks; ++nb)
        for (int cw = 2; cw <= 4; cw += 2) {
            const int tile = 16 * nb * cw;
            const int ncol = (cols + tile - 1) / tile * tile;
            const double cost = (double)(ncol / (16 * nb)) * step_cycles(nb, cw);
            if (ncol <= ld && cost < best_cost) {
                best_cost = cost;
                best.nb = nb;
                best.cw = cw;
                best.ncol = ncol;
            }
        }
    return best;
}

namespace {
// Cycles of a build, for one workgroup per CU and round: the k-steps of its
// workgroups, a few microseconds of ramp per round of resident workgroups, and
// with several segments the sum over them (about 2.4 TB/s and a launch).
double build_cycles(const KF64Plan& p, int rows, int ngp) {
    const int wg_rows = 16 * (4 / p.cw);
    const double wgs = (double)((rows + wg_rows - 1) / wg_rows) * (p.ncol / (16 * p.nb * p.cw)) * p.nseg;
    const double per_cu = (double)(long)((wgs + kCus - 1) / kCus);
    const int res = resident(p.nb);
    const double rounds = (double)(long)((per_cu + res - 1) / res);
    double c = per_cu * (p.seg_len / 4) * step_cycles(p.nb, p.cw) + rounds * 6000.0;
    if (per_cu < 2.0 && res > 1) c *= 1.25;   // a single wave per SIMD waits for its loads
    if (p.nseg > 1) c += 8000.0 + 1e-3 * 24.0 * rows * (double)p.ncol * p.nseg;
    return c;
}
}  // namespace

KF64Plan kf64_segments(KF64Plan p, int rows, int ngp, int max_seg) {
    KF64Plan best = p;
    double best_cycles = 1e300;
    for (int want = 1; want <= std::max(1, max_seg); ++want) {
        p.seg_len = ((ngp + want - 1) / want + kKSegQuant - 1) / kKSegQuant * kKSegQuant;
        p.nseg = (ngp + p.seg_len - 1) / p.seg_len;    // every segment starts inside the grid
        const double c = build_cycles(p, rows, ngp);
        if (c < best_cycles) {
            best_cycles = c;
            best = p;
        }
    }
    return best;
}

KF64Plan kf64_plan(int cols, int ld, int rows, int ngp, int max_seg, size_t max_bytes) {
    KF64Plan best{0, 0, 0, 0, 0};
    double best_cycles = 1e300;
    for (int nb = 1; nb <= kMaxBlocks; ++nb)
        for (int cw = 2; cw <= 4; cw += 2) {
            const int tile = 16 * nb * cw;
            KF64Plan p{nb, cw, (cols + tile - 1) / tile * tile, 1, ngp};
            if (p.ncol > ld) continue;
            const size_t fit = max_bytes / ((size_t)3 * rows * p.ncol * sizeof(double));
            p = kf64_segments(p, rows, ngp, (int)std::min<size_t>(max_seg, fit));
            const double c = build_cycles(p, rows, ngp);
            if (c < best_cycles) {
                best_cycles = c;
                best = p;
            }
        }
    return best;
}

size_t kf64_part_bytes(const KF64Plan& p, int rows) {
    return p.nseg > 1 ? (size_t)p.nseg * 3 * rows * p.ncol * sizeof(double) : 0;
}

namespace {

template <int KIND, int NB, int CW>
hipError_t launch(const d4* pos, const double* rho, int ld, int ngp, int g0, int rows, const JasDev& J,
                  const KF64Plan& p, double* out, int ldo, hipStream_t st) {
    constexpr int kRows = 16 * (4 / CW);
    const int n_rt = (rows + kRows - 1) / kRows;
    const int n_ct = p.ncol / (16 * NB * CW);
    hipLaunchKernelGGL((k_build_K_f64<KIND, NB, CW>), dim3((unsigned)((long)n_rt * n_ct), (unsigned)p.nseg), dim3(256),
                       0, st, pos, rho, ld, ngp, g0, rows, n_rt, p.seg_len, J, out, ldo, p.ncol);
    return hipGetLastError();
}

template <int KIND, int CW>
hipError_t launch_nb(const d4* pos, const double* rho, int ld, int ngp, int g0, int rows, const JasDev& J,
                     const KF64Plan& p, double* out, int ldo, hipStream_t st) {
    switch (p.nb) {
        case 1: return launch<KIND, 1, CW>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
        case 2: return launch<KIND, 2, CW>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
        case 3: return launch<KIND, 3, CW>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
        case 4: return launch<KIND, 4, CW>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
        case 5: return launch<KIND, 5, CW>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
        case 6: return launch<KIND, 6, CW>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
        case 7: return launch<KIND, 7, CW>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t kf64_build(const d4* pos, const double* rho, int ld, int ngp, int g0, int rows, const JasDev& J,
                      const KF64Plan& p, double* out, int ldo, hipStream_t st) {
    // the kernel assumes whole column tiles, whole stages and a grid of whole stages
    if (rows < 1 || ld < 16 || ld % 16 || (p.nseg == 1 ? ldo < p.ncol : ldo != p.ncol) || p.seg_len % kKSegQuant ||
        ngp % kKSegQuant || (long)(p.nseg - 1) * p.seg_len >= ngp || (p.cw != 2 && p.cw != 4) ||
        p.ncol % (16 * p.nb * p.cw))
        return hipErrorInvalidValue;
    if (J.kind == 0)
        return p.cw == 2 ? launch_nb<0, 2>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st)
                         : launch_nb<0, 4>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
    return p.cw == 2 ? launch_nb<1, 2>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st)
                     : launch_nb<1, 4>(pos, rho, ld, ngp, g0, rows, J, p, out, ldo, st);
}

}  // namespace xtc
