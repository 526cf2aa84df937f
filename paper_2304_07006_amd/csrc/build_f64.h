// Host interface of the FP64 K build (kernels_build_f64.h; built in its own
// translation unit, build_f64.hip, so that its MFMA accumulators live in the
// accumulation registers).
#pragma once
#include <hip/hip_runtime.h>

#include "xtc_device.h"

namespace xtc {

// How a K build over `cols` pair columns and `rows` grid rows is laid out: nb
// 16-column blocks per wave, cw waves that share their rows' generated d^x,
// ncol = cols rounded up to whole column tiles, nseg segments of seg_len
// points (a multiple of 64) of the sum over g'.
struct KF64Plan {
    int nb, cw, ncol, nseg, seg_len;
};

// The column tiling alone (nseg = 1): the shape whose MFMA and generation
// work per useful column is least, with ncol <= ld.
KF64Plan kf64_columns(int cols, int ld);

// The whole plan for rows x cols outputs and ngp points: at most max_seg
// segments, and only as many as have partials within max_bytes.
KF64Plan kf64_plan(int cols, int ld, int rows, int ngp, int max_seg, size_t max_bytes);

// Bytes of a plan's segment partials (0 with one segment: none).
size_t kf64_part_bytes(const KF64Plan& p, int rows);

// The segments of an already tiled build (nb, cw, ncol of p are kept).
KF64Plan kf64_segments(KF64Plan p, int rows, int ngp, int max_seg);

// K^x_P(g) of rows [g0, g0 + rows) against rho [ngp][ld]: out[x][r][ldo] with
// zeros in the columns [ncol, ldo) if nseg == 1, else the partials
// out[seg][x][r][ncol].  ncol may exceed ld (the occupied pairs, whose rows are
// packed to 16 columns): the columns from ld on then hold sums of other bits,
// and up to ncol - ld doubles behind the last row of rho are read, which the
// caller provides.  Returns the launch status.
hipError_t kf64_build(const d4* pos, const double* rho, int ld, int ngp, int g0, int rows, const JasDev& J,
                      const KF64Plan& p, double* out, int ldo, hipStream_t st);

}  // namespace xtc
