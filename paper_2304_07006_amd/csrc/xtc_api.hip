// libxtc: C ABI (include/xtc.h) over the gfx950 kernels.
//
// Host side only validates, lays out the caller's workspace and launches.
// Workspace layout (all offsets 256-byte aligned), for ldP = xtc_pair_ld(N)
// and ngp = Ng rounded up to 128:
//   pos    [ngp] x 4 doubles          grid positions (x, y, z, 0)
//   rho    [ngp][ldP] doubles         weighted pair densities, zero padded
//   rho_lp [NS][ngp/8][ldL][8]        reduced-precision rho (k8-packed), prec != FP64
//   rho_occ[ngp][ldO], colmap[ldO]    FP64 rho of the occupied-occupied pairs
//   stg, amax                         digit stage blocks and per-pair largest |rho|
//                                     of the integer occupied block (occ_i8.h)
//   M      [ldP][ldP] doubles         FP64 accumulator of the two-body term
//   h1acc  [ldP] doubles              FP64 accumulator of the one-body term
//   T1     [kT1Split][ldP] doubles    per-split partials (one-body, term 1)
//   E      [kESplit][N][N] doubles    per-split partials (one-body, exchange)
// with XTC_WITH_BACKWARD in prec (the adjoint reuses M for Gbar):
//   gacc [16], occw [N] f64, kidx [N],
//   reduced forms: rhoR (split rho: FP32 row-major [1][ngp][ldP], split BF16
//   k-packed [NS][ldP/8][ngp][8]), split-BF16 3-product form: GsL (k-packed
//   split Gbar, [2][ldP/8][ldP][8])
// with XTC_WITH_TC2 (two-body TC integrals; ldN = N^2 rounded up to 128):
//   Atc [ldP][ldP], Btc [ldN][ldP] FP64 accumulators
// All of that has one place for every call on a workspace.  What follows is laid
// out by each call for its own number of rows (`crows`, a multiple of 32):
//   Kc     [3][crows][ldP] doubles    K of a chunk of the adjoint
//   Ftc    [crows][ldP] doubles       F of the TC integrals
//   S      [crows][8] doubles         per-point scalars of the chunk
//   D      [4][crows][ldP] doubles    A, Bx, By, Bz of the chunk
//   Rg     [3][crows][ldN] doubles    w phi grad phi (TC integrals, FP64 form)
//   CDlp   [8][NS][crows/8][ldL][8]   C and D of the chunk, k8-packed (prec != FP64)
//   scratch: from there to the K build's part
//   K build's part: the last kres bytes (a function of the workspace alone).
// S and D are the only ones that outlive a call: xtc_contract_2body leaves them
// to an xtc_contract_1body_0body with XTC_REUSE_INTERMEDIATES on the same rows,
// with no call in between.  The K build keeps its segment partials (Kpart
// [nsegK][3][kcap][ldL] f32, then those of the occupied block; or FP64 ones) in
// its own part, so that it may run beside the contraction of another chunk.  The
// two-body products' partials (Mpart: [group][4][ldL][ldL] f32, or FP64 ones),
// those of term 1 of the one-body sum and V2's packed sums take the scratch; and
// the adjoint, which has no two-body products, keeps
//   Y [7][crows][ldP], T [crows][3][N][nocc], Wbar [crows][3],
//   gpart [ceil(crows/32) * ngp/128][16], KbL [7][NS][crows * ldP] (split operands
//   of the chunk, in rhoR's two layouts)
// there.
// ldL = ldP rounded up to 512.  The chunk capacity `cap` is the largest multiple
// of 32 rows whose buffers fit in the bytes the caller passes (layout_bytes).
// Segment partials beyond the least that a product needs only make it faster:
// xtc_workspace_size adds what the launch plans would use (plan_extra), and a
// smaller workspace, or a chunk longer than it was sized for, gets plans with
// fewer segments.
// The segment partials of the reduced forms are bounded: the K build runs over a
// chunk in equal row pieces of at most kcap rows (kcap = min(crows, the multiple
// of 1024 rows whose partials fit kKpartBudget bytes, at least 1024)), and the
// two-body GEMM over groups of row segments, each piece reduced into its FP64
// result before the next one reuses the partial buffer.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/xtc.h"
#include "build_f64.h"
#include "kernels_contract.h"
#include "kernels_fc.h"
#include "kernels_gemm_f64.h"
#include "kernels_tc2.h"
#include "kernels_lp.h"
#include "kernels_bwd.h"
#include "kernels_lowdin.h"
#include "kernels_prepare.h"
#include "occ_i8.h"

using namespace xtc;

namespace {

thread_local std::string g_err;

xtc_status fail(xtc_status st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
xtc_status fail(xtc_status st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

constexpr int kT1Split = 64, kT1SplitMax = 256;   // row splits of term 1 (one-body): in T1, and in the scratch
constexpr int kESplitMax = 256;
constexpr size_t kAlign = 256;
constexpr int kMaxN = 256;
// Grid points: kernels index the padded grid with 32-bit integers; 2^28 points
// of even one orbital pair already take 275 GB for rho alone.
constexpr int kMaxNg = 1 << 28;
constexpr size_t kLdsMax = 160 * 1024;
// The kernels that stage the occupied columns in dynamic LDS (nocc N of
// (rho, Kx, Ky, Kz)) also keep a few static reduction slots (at most 96 B);
// a workgroup's static plus dynamic LDS must fit kLdsMax.
constexpr size_t kLdsStaticReserve = 1024;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int pair_ld(int N) {
    const long npair = (long)N * (N + 1) / 2;
    return (int)((npair + kPairTile - 1) / kPairTile * kPairTile);
}

// FP32 accumulation segments of the reduced-precision forms (the partials are
// summed in FP64): g' per segment of the K build, grid rows per segment of the
// two-body GEMM.  The split-BF16 forms' error is their dropped products, so
// long segments cost nothing there; the FP32 form's error grows with the
// segment (one rounding per 4 products in v_mfma_f32_16x16x4_f32) and at
// N=128, Ng=150 000 needs 8x and 4x shorter ones to meet the 1e-6 Eh bars.
constexpr int kSegK = 8192, kSegKF32 = 1024;
constexpr int kSegM = 2048, kSegMF32 = 512;
constexpr int kRowQuant = 32;
constexpr int kOccSegMax = 32;  // most segments of the FP64 occupied-block sum over g'
constexpr size_t kKpartBudget = (size_t)16 << 30;  // bytes of K-build segment partials
constexpr int kKpartQuant = 1024;                  // rows: 32 row tiles, one XCD's resident set
// Row segments per two-body GEMM launch: two, and for smaller matrices as many
// (up to kMSegGroupMax) as fit the scratch and kMpartBudget bytes, so that a launch
// has rounds enough of workgroups (N=48 in FP32, 4000 rows: four launches of 400
// workgroups, the second round of each half empty, 173 us each; one of 1600
// takes 654).
constexpr int kMSegGroup = 2, kMSegGroupMax = 16;
constexpr size_t kMpartBudget = (size_t)512 << 20;
// Row-split FP64 products: most row segments, and bytes of their partials (a
// matrix too large for two partials has tiles enough to fill the chip).
constexpr int kTnSplitMax = 64;
constexpr size_t kMpartF64Budget = (size_t)192 << 20;
// FP64 K build of a grid too small to fill the chip: most segments of the sum
// over g', and bytes of their partials.
constexpr int kKSplitMax = 16;
constexpr size_t kKpartF64Budget = (size_t)192 << 20;
constexpr int kCus = 256;                          // compute units of an MI355X (launch shapes only)

struct Layout {
    int N, Ng, nocc, ldP, ngp, Npair, prec;
    int form, ns, es, ldL, ldO, nOP, nsegK, nspin, ldN, segK, segM;
    KF64Plan occ64;      // column tiling of the FP64 occupied block (ldO: the pairs rounded up to 16)
    int nY;              // adjoint Y slots: Cbar (3), then Abar, Bbar (4) per spin channel
    OccI8Plan i8;        // column tiling of the integer occupied block
    bool i8ok;           // one column group and the grid fits its int32 segments (else the FP64 block serves)
    int ldK8;            // row stride of its segment partials (16 i8.nct8)
    bool tc2;
    bool bwd;
    size_t pos, rho, rho_lp, rho_occ, colmap, stg, amax, M, h1acc, T1, E, e_end, gacc, occw, kidx, rhoR, GsL, Atc, Btc, GT;
    size_t fixed;        // bytes of everything that does not scale with the chunk rows (plus reserves)
    size_t chunk0;       // offset of the first chunk buffer (Kc)
    size_t per_row;      // bytes per chunk row (without the K-build partials)
    size_t kpart_row;    // bytes per row of the K-build partials (reduced forms)
    int kcap_max;        // most rows of one K-build piece
    int cap;             // chunk rows that fit (multiple of kRowQuant)
    int crows;           // rows of this call's chunk buffers
    int kcap;            // rows of the K-build partial buffer: min(crows, kcap_max)
    size_t mslab;        // bytes of the two-body partials of one segM-row segment
    size_t cdw;          // packed operand elements per row and split (CDlp)
    size_t kres;         // bytes of the K build's part
    size_t Kc, Ftc, S, D, Rg, CDlp, scr, Y, T, Wbar, gpart, KbL, kpart, end;
};

int form_of(int prec) {
    prec &= 0xF;
    return prec == XTC_FP32 ? 1 : prec == XTC_BF16X3 ? 3 : prec == XTC_BF16X6 ? 6 : 0;
}

// The FP64 K build's plan for `rows` rows with `bytes` of partials.
KF64Plan plan_build_f64(const Layout& L, int rows, size_t bytes) {
    // the budget in whole rows of kKSplitMax segments of ldP columns
    const size_t row = (size_t)kKSplitMax * 3 * L.ldP * sizeof(double);
    const size_t most = kKpartF64Budget / row * kKSplitMax / rows;
    return kf64_plan(L.Npair, L.ldP, rows, L.ngp, (int)std::min<size_t>(most, kKSplitMax), bytes);
}

Layout make_layout(const xtc_problem* pb, int prec) {
    Layout L{};
    L.N = pb->N;
    L.Ng = pb->Ng;
    L.nocc = pb->nocc;
    L.nspin = pb->occ_n_beta ? 2 : 1;
    L.prec = prec;
    L.ldP = pair_ld(pb->N);
    L.Npair = pb->N * (pb->N + 1) / 2;
    L.ngp = (int)align_up((size_t)pb->Ng, kGridPad);
    L.form = form_of(prec);
    L.ns = L.form == 1 ? 1 : L.form == 3 ? 2 : L.form == 6 ? 3 : 0;
    L.es = L.form == 1 ? 4 : 2;
    L.ldL = (int)align_up((size_t)L.ldP, kLpCols);
    L.nOP = pb->nocc * (pb->nocc + 1) / 2;
    L.occ64 = kf64_columns(L.nOP, 1 << 30);
    L.ldO = (int)align_up((size_t)L.nOP, 16);
    L.i8 = occ_i8_plan(L.nOP);
    // the integer block serves one column group (at most 144 occupied pairs).
    // Larger sets keep the FP64 block, the more accurate of the two (N=160, 20
    // occupied, 250 000 points: E0 7e-15 Eh from the oracle against 4.7e-11),
    // although two groups of the integer one would take less time (12 500 rows,
    // 100 000 points: 18.6 against 26.9 ms Pade, 21.4 against 27.0 power)
    L.i8ok = L.ngp <= occ_i8_max_points(kOccSegMax) && L.i8.groups == 1;
    L.ldK8 = 16 * L.i8.nct8;
    L.segK = L.form == 1 ? kSegKF32 : kSegK;
    L.segM = L.form == 1 ? kSegMF32 : kSegM;
    L.nsegK = (L.ngp + L.segK - 1) / L.segK;
    L.bwd = (prec & XTC_WITH_BACKWARD) != 0;
    L.tc2 = (prec & XTC_WITH_TC2) != 0;
    L.nY = 3 + 4 * L.nspin;
    L.ldN = (int)align_up((size_t)pb->N * pb->N, 128);
    const bool lp = L.form != 0;
    size_t off = 0;
    L.pos = off;     off = align_up(off + (size_t)L.ngp * 4 * sizeof(double), kAlign);
    L.rho = off;     off = align_up(off + (size_t)L.ngp * L.ldP * sizeof(double), kAlign);
    L.rho_lp = off;  off = align_up(off + (lp ? (size_t)L.ns * L.ngp * L.ldL * L.es : 0), kAlign);
    L.rho_occ = off; off = align_up(off + (lp ? (size_t)L.ngp * L.ldO * sizeof(double) : 0), kAlign);
    L.colmap = off;  off = align_up(off + (lp ? (size_t)L.ldO * sizeof(int) : 0), kAlign);
    const bool i8 = lp && L.i8ok;
    L.stg = off;     off = align_up(off + (i8 ? occ_i8_stage_bytes(L.i8, L.ngp) : 0), kAlign);
    L.amax = off;    off = align_up(off + (i8 ? (size_t)L.ldK8 * sizeof(double) : 0), kAlign);
    L.M = off;       off = align_up(off + (size_t)L.nspin * L.ldP * L.ldP * sizeof(double), kAlign);
    L.h1acc = off;   off = align_up(off + (size_t)L.nspin * L.ldP * sizeof(double), kAlign);
    L.T1 = off;      off = align_up(off + (size_t)kT1Split * L.ldP * sizeof(double), kAlign);
    L.E = off;       off = align_up(off + (size_t)kESplitMax * L.N * L.N * sizeof(double), kAlign);
    L.e_end = off;
    L.gacc = off;    off = align_up(off + (L.bwd ? kGradMax * sizeof(double) : 0), kAlign);
    L.occw = off;    off = align_up(off + (L.bwd ? (size_t)3 * L.N * sizeof(double) : 0), kAlign);
    L.kidx = off;    off = align_up(off + (L.bwd ? (size_t)L.N * sizeof(int) : 0), kAlign);
    L.rhoR = off;    off = align_up(off + (L.bwd && lp ? (size_t)L.ns * L.ngp * L.ldP * L.es : 0), kAlign);
    const bool bsplit = L.bwd && L.form == 3;   // split-BF16 X Gbar products (3-product form)
    // open shell: Gbar^a, Gbar^b in M, their transposes in GT; split copies
    // (k-packed) of Gbar (closed) or of Gbar^a, Gbar^b, Gbar^aT, Gbar^bT
    L.GT = off;      off = align_up(off + (L.bwd && L.nspin == 2 ? (size_t)2 * L.ldP * L.ldP * sizeof(double) : 0),
                                    kAlign);
    L.GsL = off;     off = align_up(off + (bsplit ? (size_t)(L.nspin == 2 ? 4 : 1) * L.ns * L.ldP * L.ldP * L.es : 0),
                                    kAlign);
    L.Atc = off;     off = align_up(off + (L.tc2 ? (size_t)L.ldP * L.ldP * sizeof(double) : 0), kAlign);
    L.Btc = off;     off = align_up(off + (L.tc2 ? (size_t)L.ldN * L.ldP * sizeof(double) : 0), kAlign);
    const size_t gslab = (size_t)(L.ngp / 128) * kGradMax * sizeof(double);   // one 32-row tile of partials
    // partials of one row segment: the four components of the two-body GEMM, or
    // the TC integrals' B (three components summed in one partial)
    L.mslab = lp ? std::max((size_t)4 * L.ldL * L.ldL, L.tc2 ? (size_t)L.ldN * L.ldL : 0) * sizeof(float) : 0;
    // packed operands: C and D of the two-body GEMM (8 components of ldL), or
    // w phi grad phi (3 of ldN) and K (3 of ldL) of the TC integrals
    L.cdw = std::max((size_t)8 * L.ldL, L.tc2 ? (size_t)3 * L.ldN + (size_t)3 * L.ldL : 0);
    L.chunk0 = off;
    L.fixed = off + (lp ? (size_t)kMSegGroup * L.mslab : 0) + (L.bwd ? gslab : 0) + 16 * kAlign;
    L.per_row = (size_t)L.nspin * (8 * sizeof(double) + (size_t)4 * L.ldP * sizeof(double));
    if (lp) L.per_row += (size_t)kOccSegMax * 3 * std::max(L.ldO, L.ldK8) * sizeof(double);
    if (lp) L.per_row += L.cdw * L.ns * L.es;
    L.kpart_row = lp ? (size_t)L.nsegK * 3 * L.ldL * sizeof(float) : 0;
    L.kcap_max = lp ? (int)std::max<size_t>(kKpartQuant, kKpartBudget / L.kpart_row / kKpartQuant * kKpartQuant) : 0;
    if (L.tc2) L.per_row += (size_t)L.ldP * sizeof(double) + (lp ? 0 : (size_t)3 * L.ldN * sizeof(double));
    if (L.bwd)
        L.per_row += (size_t)(3 + L.nY) * L.ldP * sizeof(double) + (size_t)3 * L.N * L.nocc * sizeof(double) +
                     3 * sizeof(double) + (gslab + 31) / 32 + (lp ? (size_t)7 * L.ns * L.ldP * L.es : 0);
    L.cap = 0;
    return L;
}

// Most bytes of K-build partials that FP64 plans of 512 rows and more ask for
// (fewer rows split their sums as far as that goes): the largest over rows a
// factor 0.7 apart, and 1.3 of that for those between them.  A function of N and
// Ng alone, for every call on a workspace; the plans take 3 us each, so a thread
// keeps its last result (passes of eight 190-row chunks at N=12: 426 -> 391 us).
size_t most_build_partials(const Layout& L) {
    thread_local int last_N = 0, last_Ng = 0;
    thread_local size_t last = 0;
    if (L.N == last_N && L.Ng == last_Ng) return last;
    size_t most = 0;
    for (double rows = L.Ng; rows == L.Ng || rows >= 512; rows *= 0.7)
        most = std::max(most, kf64_part_bytes(plan_build_f64(L, (int)rows, (size_t)1 << 62), (int)rows));
    last = align_up(std::min(most + most / 10 * 3, kKpartF64Budget), kAlign);
    last_N = L.N;
    last_Ng = L.Ng;
    return last;
}

// Bytes that the buffers of a chunk of `rows` rows (a multiple of kRowQuant)
// need, without the partials that only make it faster.
size_t layout_bytes(const Layout& L, size_t rows) {
    return L.fixed + rows * L.per_row + std::min(rows, (size_t)L.kcap_max) * L.kpart_row;
}

// Chunk capacity that `bytes` allows (the inverse of layout_bytes).
long chunk_capacity(const Layout& L, size_t bytes) {
    if (bytes <= L.fixed) return 0;
    const size_t b = bytes - L.fixed;
    size_t cap = b / (L.per_row + L.kpart_row);            // rows, if the partials cover all of them
    if (L.kpart_row > 0 && cap > (size_t)L.kcap_max) cap = (b - (size_t)L.kcap_max * L.kpart_row) / L.per_row;
    return std::min((long)std::min<size_t>(cap, kMaxNg) / kRowQuant * kRowQuant,
                    (long)align_up((size_t)L.Ng, kRowQuant));
}

// The capacity, and the offsets of the chunk buffers of a call on `rows` rows (at
// most the capacity).
void place_chunk(Layout& L, size_t bytes, long rows) {
    const bool lp = L.form != 0, b = L.bwd;
    const size_t gslab = (size_t)(L.ngp / 128) * kGradMax * sizeof(double);
    L.cap = (int)chunk_capacity(L, bytes);
    L.end = bytes / kAlign * kAlign;
    const auto place = [&](size_t n) {
        size_t off = L.chunk0;
        L.Kc = off;      off = align_up(off + (b ? 3 * n * L.ldP * sizeof(double) : 0), kAlign);
        L.Ftc = off;     off = align_up(off + (L.tc2 ? n * L.ldP * sizeof(double) : 0), kAlign);
        L.S = off;       off = align_up(off + L.nspin * n * 8 * sizeof(double), kAlign);
        L.D = off;       off = align_up(off + L.nspin * 4 * n * L.ldP * sizeof(double), kAlign);
        L.Rg = off;      off = align_up(off + (L.tc2 && !lp ? 3 * n * L.ldN * sizeof(double) : 0), kAlign);
        L.CDlp = off;    off = align_up(off + (lp ? L.cdw * L.ns * n * L.es : 0), kAlign);
        L.scr = off;
        L.Y = off;       off = align_up(off + (b ? L.nY * n * L.ldP * sizeof(double) : 0), kAlign);
        L.T = off;       off = align_up(off + (b ? n * 3 * L.N * L.nocc * sizeof(double) : 0), kAlign);
        L.Wbar = off;    off = align_up(off + (b ? n * 3 * sizeof(double) : 0), kAlign);
        L.gpart = off;   off = align_up(off + (b ? (n + 31) / 32 * gslab : 0), kAlign);
        L.KbL = off;     off = align_up(off + (b && lp ? 7 * L.ns * n * L.ldP * L.es : 0), kAlign);
        return off;
    };
    // the K build's part.  Reduced forms: its partials for a chunk of the capacity,
    // and those of the occupied block after them in time.  FP64: what plans ask for,
    // if the call's rows fit beside it; with the adjoint's buffers half of those,
    // which are dead while K is built.
    const size_t cap = (size_t)L.cap, full = place(cap);
    if (lp)
        L.kres = align_up(std::max(std::min(cap, (size_t)L.kcap_max) * L.kpart_row,
                                   (size_t)kOccSegMax * 3 * cap * std::max(L.ldO, L.ldK8) * sizeof(double)), kAlign);
    else if (b)
        L.kres = std::min(most_build_partials(L), (L.end > L.scr ? L.end - L.scr : 0) / 2 / kAlign * kAlign);
    else if (const size_t k = most_build_partials(L))
        L.kres = bytes > k && rows <= chunk_capacity(L, bytes - k) ? k : 0;
    if (std::max(full, L.scr + (lp ? (size_t)kMSegGroup * L.mslab : 0)) + (lp ? L.kres : 0) > L.end)
        L.cap = 0;   // cannot happen by construction; refuse rather than overrun
    const size_t n = std::min(cap, align_up((size_t)std::max(rows, 1L), kRowQuant));
    place(n);
    L.crows = (int)n;
    L.kcap = std::min(L.crows, L.kcap_max);
    L.kpart = L.end - L.kres;
}

// Bytes for the segment partials of a K build (from kpart on), and for those of
// the two-body products, the one-body sums and V2 (from scr on).
size_t build_bytes(const Layout& L) { return L.kres; }
size_t scratch_bytes(const Layout& L) { return L.kpart - L.scr; }

xtc_status check_problem(const xtc_problem* pb) {
    if (!pb) return fail(XTC_E_ARG, "problem is NULL");
    if (pb->reserved != 0) return fail(XTC_E_ARG, "problem.reserved must be 0");
    if (pb->N < 1 || pb->N > kMaxN) return fail(XTC_E_ARG, "N=%d outside [1,%d]", pb->N, kMaxN);
    if (pb->Ng < 1) return fail(XTC_E_ARG, "Ng=%d < 1", pb->Ng);
    if (pb->Ng > kMaxNg) return fail(XTC_E_UNSUPPORTED, "Ng=%d above %d", pb->Ng, kMaxNg);
    if (pb->nocc < 1 || pb->nocc > pb->N || pb->nocc > kMaxOcc)
        return fail(XTC_E_ARG, "nocc=%d outside [1,min(N,%d)]", pb->nocc, kMaxOcc);
    if (!pb->xyz || !pb->w || !pb->phi || !pb->occ) return fail(XTC_E_ARG, "NULL array in problem");
    std::vector<char> seen(pb->N, 0);
    for (int i = 0; i < pb->nocc; ++i) {
        const int k = pb->occ[i];
        if (k < 0 || k >= pb->N) return fail(XTC_E_ARG, "occ[%d]=%d outside [0,N)", i, k);
        if (seen[k]) return fail(XTC_E_ARG, "occ[%d]=%d repeated", i, k);
        seen[k] = 1;
        if (pb->occ_n && !std::isfinite(pb->occ_n[i])) return fail(XTC_E_ARG, "occ_n[%d] not finite", i);
        if (pb->occ_n_beta && !std::isfinite(pb->occ_n_beta[i]))
            return fail(XTC_E_ARG, "occ_n_beta[%d] not finite", i);
    }
    if ((size_t)pb->nocc * pb->N * 4 * sizeof(double) > kLdsMax - kLdsStaticReserve)
        return fail(XTC_E_UNSUPPORTED, "nocc*N=%d exceeds the on-chip staging of the intermediates",
                    pb->nocc * pb->N);
    return XTC_OK;
}

xtc_status check_prec(int prec) {
    const int base = prec & 0xF;
    if ((prec & ~(0xF | XTC_WITH_BACKWARD | XTC_WITH_TC2)) ||
        (base != XTC_FP64 && base != XTC_FP32 && base != XTC_BF16X3 && base != XTC_BF16X6))
        return fail(XTC_E_ARG, "prec=%d unknown", prec);
    return XTC_OK;
}

xtc_status check_jastrow(const xtc_jastrow* j, JasDev* out) {
    if (!j) return fail(XTC_E_ARG, "jastrow is NULL");
    JasDev d{};
    d.kind = j->kind;
    if (j->kind == 0) {
        if (!(std::isfinite(j->b) && j->b >= 0.0)) return fail(XTC_E_ARG, "Pade b=%g must be finite and >= 0", j->b);
        d.b = j->b;
        d.ncoef = 0;
    } else if (j->kind == 1) {
        if (j->ncoef < 1 || j->ncoef > 16) return fail(XTC_E_ARG, "ncoef=%d outside [1,16]", j->ncoef);
        for (int k = 0; k < j->ncoef; ++k) {
            if (!std::isfinite(j->coef[k])) return fail(XTC_E_ARG, "coef[%d] not finite", k);
            d.dcoef[k] = (k + 1) * j->coef[k];
            if (k >= 1) d.d2coef[k - 1] = (k + 1) * k * j->coef[k];
        }
        d.ncoef = j->ncoef;
    } else {
        return fail(XTC_E_ARG, "jastrow kind=%d unknown", j->kind);
    }
    d.fb = (float)d.b;
    for (int k = 0; k < 16; ++k) {
        d.fdcoef[k] = (float)d.dcoef[k];
        d.fd2coef[k] = (float)d.d2coef[k];
    }
    *out = d;
    return XTC_OK;
}

xtc_status check_ws(const Layout& L, void* ws, size_t bytes) {
    if (!ws) return fail(XTC_E_WORKSPACE, "workspace is NULL");
    if ((uintptr_t)ws % kAlign) return fail(XTC_E_WORKSPACE, "workspace not 256-byte aligned");
    if (L.cap < kRowQuant)
        return fail(XTC_E_WORKSPACE, "workspace of %zu bytes holds no chunk (need >= %zu)", bytes,
                    layout_bytes(L, kRowQuant));
    return XTC_OK;
}

xtc_status check_range(const Layout& L, int g0, int g1) {
    if (!(0 <= g0 && g0 < g1 && g1 <= L.Ng)) return fail(XTC_E_ARG, "rows [%d,%d) not inside [0,%d)", g0, g1, L.Ng);
    if (g1 - g0 > L.cap)
        return fail(XTC_E_WORKSPACE, "chunk of %d rows exceeds the workspace capacity of %d rows", g1 - g0, L.cap);
    return XTC_OK;
}

xtc_status check_align(const void* p, const char* name) {
    if ((uintptr_t)p % 32) return fail(XTC_E_ARG, "%s must be 32-byte aligned", name);
    return XTC_OK;
}

// Occupations of spin channel `spin` (0 alpha, 1 beta) and of the total
// density.  Closed shell (occ_n_beta NULL): one channel, total = 2 n.
OccList make_occ(const xtc_problem* pb, int spin = 0) {
    OccList o{};
    o.n = pb->nocc;
    for (int i = 0; i < pb->nocc; ++i) {
        const double na = pb->occ_n ? pb->occ_n[i] : 1.0;
        o.k[i] = pb->occ[i];
        if (pb->occ_n_beta) {
            const double nb = pb->occ_n_beta[i];
            o.w[i] = spin == 0 ? na : nb;
            o.wt[i] = na + nb;
        } else {
            o.w[i] = na;
            o.wt[i] = 2.0 * na;
        }
    }
    return o;
}

xtc_status launched(const char* what) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(XTC_E_HIP, "%s: %s", what, hipGetErrorString(e));
    return XTC_OK;
}

template <typename T>
T* at(void* ws, size_t off) { return reinterpret_cast<T*>(static_cast<char*>(ws) + off); }

xtc_status fill(double* p, size_t n, hipStream_t st) {
    if (n == 0) return XTC_OK;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_fill, dim3((unsigned)blocks), dim3(256), 0, st, p, n, 0.0);
    return launched("fill");
}

// Intermediates of rows [g0, g1) into D and S of the workspace.
xtc_status run_intermediates(const Layout& L, const xtc_problem* pb, const double* K, int g0, int g1,
                             void* ws, hipStream_t st) {
    const int rows = g1 - g0;
    const double* rho_rows = at<double>(ws, L.rho) + (size_t)g0 * L.ldP;
    const size_t dstride = (size_t)L.crows * L.ldP;
    const size_t lds = (size_t)L.nocc * L.N * 4 * sizeof(double);
    const int nb = (L.N + kITile - 1) / kITile, tiles = nb * (nb + 1) / 2;
    const int threads = std::min(256, (int)align_up((size_t)tiles, 64));
    const int blocks = std::min(rows, 16384);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_intermediates,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) {
            (void)hipGetLastError();   // do not leave the error for the caller's next HIP call
            return fail(XTC_E_HIP, "intermediates LDS attribute: %s", hipGetErrorString(e));
        }
    }
    for (int sp = 0; sp < L.nspin; ++sp) {
        const OccList occ = make_occ(pb, sp);
        double* D = at<double>(ws, L.D) + (size_t)sp * 4 * dstride;
        double* S = at<double>(ws, L.S) + (size_t)sp * L.crows * 8;
        hipLaunchKernelGGL(k_intermediates, dim3(blocks), dim3(threads), lds, st,
                           rho_rows, K, rows, L.ldP, L.N, occ, D, dstride, S);
        xtc_status s;
        if ((s = launched("intermediates")) != XTC_OK) return s;
    }
    return XTC_OK;
}

// ---------------------------------------------------------------- reduced precision
// Pack up to kPackMax FP64 row-major arrays [nrows][ld_src] into consecutive
// components (comp_stride elements apart) of the k8-packed operand format.
xtc_status pack_many(int form, const PackSrc& src, int ncomp, int nrows, int ld_src, int ncols, int n8, int ld_dst,
                     void* dst, size_t split_stride, size_t comp_stride, hipStream_t st) {
    const dim3 grid((ld_dst + 255) / 256, n8, ncomp);
    const auto kernel = form == 1 ? k_pack_lp<1> : form == 3 ? k_pack_lp<3> : k_pack_lp<6>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, src, nrows, ld_src, ncols, ld_dst, dst, split_stride,
                       comp_stride);
    return launched("pack_lp");
}

xtc_status pack_any(int form, const double* src, int nrows, int ld_src, int ncols, int n8, int ld_dst, void* dst,
                    size_t split_stride, hipStream_t st) {
    return pack_many(form, PackSrc{{src}}, 1, nrows, ld_src, ncols, n8, ld_dst, dst, split_stride, 0, st);
}

// Cycles per k-step of a workgroup of `waves` waves of which those that own some
// of `cols` columns multiply (`blocks` 16-column blocks of `block` MFMA cycles
// each per 16 rows), on four SIMDs: the active waves' MFMAs, and about 350
// cycles of generation per wave.
double lp_step_cycles(int waves, int blocks, int cols, double block) {
    const int active = std::min(waves, (cols + 16 * blocks - 1) / (16 * blocks));
    return ((active + 3) / 4) * (waves / 4) * blocks * block + (waves / 4) * 350.0;
}

// Tile variant of the reduced K build over `rows` rows: the one whose busiest
// CU needs the fewest cycles per k-step (at least 900, the latency of a step).
// 0 is the standard tile, which every grid of more than a few rounds takes; N=21
// on 1501 rows is 47 workgroups of it (91 us) and 188 of 16 x 128 columns (53
// us).
struct LpVariant {
    int waves, blocks;
};
constexpr LpVariant kLpVariants[] = {{8, 0}, {8, 2}, {4, 2}, {4, 1}};   // blocks 0: LpTile's
int lp_tile(const Layout& L, int rows, int nc, int std_blocks) {
    const double block = nc * (L.form == 1 ? 8 * 32.0 : L.form * 16.0);   // MFMA cycles of 16 rows x 16 columns
    int best = 0;
    double best_cycles = 1e300;
    for (int i = 0; i < 4; ++i) {
        const int w = kLpVariants[i].waves, nb = i ? kLpVariants[i].blocks : std_blocks;
        const int cols = w * 16 * nb;
        const int full = L.Npair / cols, rem = L.Npair - full * cols;
        const double tiles = (double)((rows + 4 * w - 1) / (4 * w)) * L.nsegK;   // workgroups per column tile
        const double step = lp_step_cycles(w, nb, cols, block), last = rem ? lp_step_cycles(w, nb, rem, block) : 0.0;
        const double busiest = std::ceil(tiles * (full + (rem ? 1 : 0)) / kCus) * (full ? step : last);
        const double cycles = std::max({900.0, std::min(busiest, tiles * (full * step + last) / kCus + step),
                                        full ? step : last});
        if (cycles < 0.8 * best_cycles) {
            best = i;
            best_cycles = cycles;
        }
    }
    return best;
}

// The pair columns [coff, ncol) in tiles of one variant.
template <int KIND, int FORM, int NC, int NW, int NB>
void launch_build_lp_tile(const Layout& L, int coff, int ncol, int g0, int rows, const JasDev& J, void* ws,
                          hipStream_t st) {
    constexpr int cols = NW * 16 * NB;
    const int n_rt = (rows + 4 * NW - 1) / (4 * NW);
    const int n_ct = (ncol - coff + cols - 1) / cols;
    hipLaunchKernelGGL((k_build_K_lp<KIND, FORM, NC, NW, NB>), dim3(n_rt * n_ct * L.nsegK), dim3(64 * NW), 0, st,
                       at<d4>(ws, L.pos), at<void>(ws, L.rho_lp), (size_t)L.ngp * L.ldL, L.ldL, L.ngp, g0, rows, n_rt,
                       L.segK, J, at<float>(ws, L.kpart), L.kcap, coff, ncol, n_ct, L.nsegK);
}

// Variant (0: standard) for a last column tile of `cols` < standard columns, by
// cycles per 32 rows and k-step: its active waves' MFMAs four waves at a time
// plus everyone's generation, against small tiles whose four waves are all
// busy.  N=64 ends in 32 pairs of a 512-column tile, N=96 in 48: 5.81 -> 5.53
// ms for 5000 rows and 40 000 points, 31.8 -> 30.8 ms for 100 000.
int lp_remainder(const Layout& L, int cols, int nc, int std_blocks) {
    const double block = nc * (L.form == 1 ? 8 * 32.0 : L.form * 16.0);   // MFMA cycles of 16 rows x 16 columns
    const int active = (cols + 16 * std_blocks - 1) / (16 * std_blocks);
    double best_cycles = 0.85 * (((active + 3) / 4) * 2 * std_blocks * block + 700.0);
    int best = 0;
    for (int i = 2; i < 4; ++i) {
        const int nb = kLpVariants[i].blocks;
        const double c = 2.0 * ((cols + 64 * nb - 1) / (64 * nb)) * (nb * block + 350.0);
        if (c < best_cycles) {
            best = i;
            best_cycles = c;
        }
    }
    return best;
}

template <int KIND, int FORM, int NC>
void launch_build_lp(const Layout& L, int g0, int rows, const JasDev& J, void* ws, hipStream_t st) {
    typedef LpTile<KIND, FORM, NC> Std;
    constexpr int cols = Std::NW * 16 * Std::NB;
    const auto part = [&](int variant, int coff, int ncol) {   // columns from Npair on are not read
        switch (variant) {
            case 0: return launch_build_lp_tile<KIND, FORM, NC, Std::NW, Std::NB>(L, coff, ncol, g0, rows, J, ws, st);
            case 1: return launch_build_lp_tile<KIND, FORM, NC, 8, 2>(L, coff, ncol, g0, rows, J, ws, st);
            case 2: return launch_build_lp_tile<KIND, FORM, NC, 4, 2>(L, coff, ncol, g0, rows, J, ws, st);
            default: return launch_build_lp_tile<KIND, FORM, NC, 4, 1>(L, coff, ncol, g0, rows, J, ws, st);
        }
    };
    const int variant = lp_tile(L, rows, NC, Std::NB);
    const int full = L.Npair / cols * cols, rem = L.Npair - full;
    // (a second launch runs after the first: not worth it within a few rounds)
    const long wgs = (long)((rows + 4 * Std::NW - 1) / (4 * Std::NW)) * (full / cols) * L.nsegK;
    const int last = variant == 0 && rem > 0 && wgs >= 4 * kCus ? lp_remainder(L, rem, NC, Std::NB) : 0;
    if (last == 0) return part(variant, 0, L.Npair);
    part(0, 0, full);
    part(last, full, L.Npair);
}

// The split K build of rows [g0, g0 + rows) (nc = 3: K, or nc = 1: F of the
// TC integrals) in equal pieces (multiples of 32 rows) of at most kcap rows:
// segment partials, then their FP64 sum into out[c][r][P] (component stride
// `rows` rows).  Each piece costs about a millisecond of launch ramp and tail
// at N=160, so the pieces are as few as the partial buffer allows.
template <int NC>
xtc_status build_lp_pieces(const Layout& L, int g0, int rows, const JasDev& J, double* out, void* ws, hipStream_t st) {
    xtc_status s;
    const int npiece = (rows + L.kcap - 1) / L.kcap;
    const int piece = std::min(L.kcap, (int)align_up((size_t)((rows + npiece - 1) / npiece), kRowQuant));
    for (int r0 = 0; r0 < rows; r0 += piece) {
        const int nr = std::min(piece, rows - r0);
        if (J.kind == 0) {
            if (L.form == 1) launch_build_lp<0, 1, NC>(L, g0 + r0, nr, J, ws, st);
            else if (L.form == 3) launch_build_lp<0, 3, NC>(L, g0 + r0, nr, J, ws, st);
            else launch_build_lp<0, 6, NC>(L, g0 + r0, nr, J, ws, st);
        } else {
            if (L.form == 1) launch_build_lp<1, 1, NC>(L, g0 + r0, nr, J, ws, st);
            else if (L.form == 3) launch_build_lp<1, 3, NC>(L, g0 + r0, nr, J, ws, st);
            else launch_build_lp<1, 6, NC>(L, g0 + r0, nr, J, ws, st);
        }
        if ((s = launched(NC == 3 ? "build_K_lp" : "build_F_lp")) != XTC_OK) return s;
        const size_t n4 = (size_t)NC * nr * L.ldP / 4;   // k_reduce_K: four pairs per thread
        const unsigned blocks = (unsigned)std::min<size_t>((n4 + 255) / 256, 16384);
        hipLaunchKernelGGL(k_reduce_K, dim3(blocks), dim3(256), 0, st, at<float>(ws, L.kpart), L.nsegK, L.kcap,
                           L.ldL, nr, L.ldP, L.Npair, out + (size_t)r0 * L.ldP, rows, NC);
        if ((s = launched("reduce_K")) != XTC_OK) return s;
    }
    return XTC_OK;
}

// How the occupied-occupied pairs of K are computed in the reduced forms.
enum OccMode {
    kOccReduced = 0,   // left in the reduced arithmetic (XTC_K_REDUCED_OCC)
    kOccExact = 1,     // integer-sliced block if the grid fits it, else FP64 MFMA
    kOccFP64 = 2       // FP64 MFMA block (XTC_K_OCC_FP64)
};

xtc_status build_K_lp(const Layout& L, int g0, int rows, const JasDev& J, double* K, int occ, void* ws,
                      hipStream_t st) {
    xtc_status s;
    if ((s = build_lp_pieces<3>(L, g0, rows, J, K, ws, st)) != XTC_OK) return s;
    if (occ == kOccReduced) return XTC_OK;
    // occupied-occupied pairs, written over the reduced-precision values:
    // segments of the sum over g' (enough, and evenly enough, to fill the chip),
    // FP64 partials, then a fixed-order reduction scattered into K
    double* part = at<double>(ws, L.kpart);
    int nseg = 0, ldK = L.occ64.ncol;
    if (occ == kOccExact && L.i8ok && occ_i8_dscale(J) > 0.0) {
        ldK = L.ldK8;
        nseg = occ_i8_build(at<d4>(ws, L.pos), at<void>(ws, L.stg), L.i8, L.ngp, g0, rows, J,
                            at<unsigned long long>(ws, L.amax), part, ldK, kOccSegMax, st);
        if (nseg == 0) {
            const hipError_t e = hipGetLastError();   // 0 segments without a HIP error: a layout check failed
            return e != hipSuccess ? fail(XTC_E_HIP, "integer occupied block: %s", hipGetErrorString(e))
                                   : fail(XTC_E_UNSUPPORTED, "integer occupied block: grid or rows outside its range");
        }
        if ((s = launched("build_K_occ_i8")) != XTC_OK) return s;
    } else {
        const size_t fit = build_bytes(L) / ((size_t)3 * rows * ldK * sizeof(double));
        const KF64Plan p = kf64_segments(L.occ64, rows, L.ngp, (int)std::min<size_t>(kOccSegMax, fit));
        nseg = p.nseg;
        const hipError_t e = kf64_build(at<d4>(ws, L.pos), at<double>(ws, L.rho_occ), L.ldO, L.ngp, g0, rows, J, p,
                                        part, ldK, st);
        if (e != hipSuccess) return fail(XTC_E_HIP, "build_K_occ_f64: %s", hipGetErrorString(e));
    }
    const size_t nel = (size_t)3 * rows * L.nOP;
    hipLaunchKernelGGL(k_reduce_occ, dim3((unsigned)std::min<size_t>((nel + 255) / 256, 8192)), dim3(256), 0, st, part,
                       nseg, rows, ldK, at<int>(ws, L.colmap), L.nOP, L.ldP, K);
    return launched("reduce_occ");
}

// part[y] = C^T D over one row segment of seg_len rows and a group of cpw of the
// ncomp components, y = group * nseg_r + segment (k_gemm_tn_lp); returns the
// number of partials written through *nparts.
xtc_status gemm_tn_lp(int form, const void* C, int ldC, size_t c_split, const void* D, int ldD, size_t d_split,
                      int rows32, int pmax, int rmax, int ncomp, int cpw, int seg_len, float* part, int* nparts,
                      hipStream_t st) {
    const int nseg_r = (rows32 + seg_len - 1) / seg_len;
    const int ny = (ncomp / cpw) * nseg_r;
    *nparts = ny;
    // few tiles: 64 x 64 outputs per workgroup, or 32 x 32 if those are still
    // fewer than CUs (N=21, 1501 rows, is one 256 x 256 tile per component: 95 -> 28 us)
    const long big = (long)((pmax + (form == 3 ? 255 : 127)) / (form == 3 ? 256 : 128)) * ((rmax + 255) / 256);
    if (big * ny < kCus / 2) {
        const int b = (long)((pmax + 63) / 64) * ((rmax + 63) / 64) * ny >= kCus ? 2 : 1;
        const int n_pt = (pmax + 32 * b - 1) / (32 * b), n_rt = (rmax + 32 * b - 1) / (32 * b);
        const auto kernel = form == 1 ? (b == 2 ? k_gemm_tn_small<1, 2, 2> : k_gemm_tn_small<1, 1, 1>)
                          : form == 3 ? (b == 2 ? k_gemm_tn_small<3, 2, 2> : k_gemm_tn_small<3, 1, 1>)
                                      : (b == 2 ? k_gemm_tn_small<6, 2, 2> : k_gemm_tn_small<6, 1, 1>);
        hipLaunchKernelGGL(kernel, dim3(n_pt * n_rt, ny), dim3(256), 0, st, C, ldC, c_split, D, ldD, d_split, rows32,
                           n_pt, cpw, seg_len, nseg_r, part);
        return launched("gemm_tn_small");
    }
    if (form == 3 && ldC % 256 == 0 && ldD % 256 == 0) {
        // both operands staged in LDS (256 x 256 tiles over [0, pmax) x [0, rmax)),
        // dealt to the 8 XCDs in ranges of per_xcd tiles
        const int n_pt = (pmax + 255) / 256, n_rt = (rmax + 255) / 256;
        const int per_xcd = (n_pt * n_rt + 7) / 8;
        const dim3 grid(8 * per_xcd, ny);
        hipLaunchKernelGGL((k_gemm_tn_lds<3>), grid, dim3(kTnThreads), 0, st, C, ldC, c_split, D, ldD, d_split, rows32,
                           n_pt, n_rt, per_xcd, pmax, rmax, cpw, seg_len, nseg_r, part);
        return launched("gemm_tn_lds");
    }
    const int n_pt = ldC / 128, n_rt = ldD / 256;
    const dim3 grid(n_pt * n_rt, ny);
    if (form == 1)
        hipLaunchKernelGGL((k_gemm_tn_lp<1>), grid, dim3(256), 0, st, C, ldC, c_split, D, ldD, d_split, rows32, n_pt,
                           pmax, rmax, cpw, seg_len, nseg_r, part);
    else if (form == 3)
        hipLaunchKernelGGL((k_gemm_tn_lp<3>), grid, dim3(256), 0, st, C, ldC, c_split, D, ldD, d_split, rows32, n_pt,
                           pmax, rmax, cpw, seg_len, nseg_r, part);
    else
        hipLaunchKernelGGL((k_gemm_tn_lp<6>), grid, dim3(256), 0, st, C, ldC, c_split, D, ldD, d_split, rows32, n_pt,
                           pmax, rmax, cpw, seg_len, nseg_r, part);
    return launched("gemm_tn_lp");
}

// M[P][R] (+)= sum of nparts partials of ldC x ldD floats, P < pmax, R < rmax.
xtc_status reduce_parts(const float* part, int nparts, int ldC, int ldD, int pmax, int rmax, double* M, int ldM,
                        int accumulate, hipStream_t st) {
    const size_t n4 = (size_t)pmax * rmax / 4;   // k_reduce_M: four R per thread
    const unsigned blocks = (unsigned)std::min<size_t>((n4 + 255) / 256, 16384);
    hipLaunchKernelGGL(k_reduce_M, dim3(blocks), dim3(256), 0, st, part, nparts, (size_t)ldC * ldD, ldD, pmax, rmax, M,
                       ldM, accumulate);
    return launched("reduce_M");
}

// Row segments per launch that `bytes` of partials allow (at least kMSegGroup).
int m_seg_group(const Layout& L, size_t bytes) {
    const size_t fit = std::min(bytes, kMpartBudget) / L.mslab;
    return (int)std::min<size_t>(kMSegGroupMax, std::max<size_t>(kMSegGroup, fit));
}

// M (+)= C^T D over rows32 packed operand rows (reduced forms), launched in
// groups of row segments of segM rows that fit the partial buffer: each group's FP32 partials
// are summed in FP64 into M before the next group reuses the partial buffer.
xtc_status gemm_tn_grouped(const Layout& L, const char* C, int ldC, size_t c_split, const char* D, int ldD,
                           size_t d_split, int rows32, int pmax, int rmax, int ncomp, int cpw, double* M, int ldM,
                           int accumulate, void* ws, hipStream_t st) {
    xtc_status s;
    float* part = at<float>(ws, L.scr);
    const int group = m_seg_group(L, scratch_bytes(L)) * L.segM;
    for (int q0 = 0; q0 < rows32; q0 += group) {
        const int nr = std::min(group, rows32 - q0);
        const size_t shift = (size_t)(q0 / 8) * 8 * L.es;   // bytes per packed row group and column
        int np = 0;
        if ((s = gemm_tn_lp(L.form, C + shift * ldC, ldC, c_split, D + shift * ldD, ldD, d_split, nr, pmax, rmax,
                            ncomp, cpw, L.segM, part, &np, st)) != XTC_OK)
            return s;
        if ((s = reduce_parts(part, np, ldC, ldD, pmax, rmax, M, ldM, q0 == 0 ? accumulate : 1, st)) != XTC_OK)
            return s;
    }
    return XTC_OK;
}

xtc_status gemm2b_lp(const Layout& L, const double* K, int g0, int rows, int accumulate, void* ws, hipStream_t st) {
    xtc_status s;
    const int rows32 = (int)align_up((size_t)rows, kRowQuant);
    const int n8 = rows32 / 8;
    const size_t split_stride = (size_t)L.crows * L.ldL;                 // elements of one split of one component
    const size_t comp_bytes = (size_t)L.ns * split_stride * L.es;
    char* cd = at<char>(ws, L.CDlp);
    const double* rho_rows = at<double>(ws, L.rho) + (size_t)g0 * L.ldP;
    const size_t ks = (size_t)rows * L.ldP, ds = (size_t)L.crows * L.ldP, comp = (size_t)L.ns * split_stride;
    if ((s = pack_many(L.form, PackSrc{{rho_rows, K, K + ks, K + 2 * ks}}, 4, rows, L.ldP, L.ldP, n8, L.ldL, cd,
                       split_stride, comp, st)) != XTC_OK)
        return s;
    // one spin channel at a time: its D into the operand buffer, GEMM, reduction into M^s
    for (int sp = 0; sp < L.nspin; ++sp) {
        const double* D = at<double>(ws, L.D) + (size_t)sp * 4 * L.crows * L.ldP;
        if ((s = pack_many(L.form, PackSrc{{D, D + ds, D + 2 * ds, D + 3 * ds}}, 4, rows, L.ldP, L.ldP, n8, L.ldL,
                           cd + 4 * comp_bytes, split_stride, comp, st)) != XTC_OK)
            return s;
        if ((s = gemm_tn_grouped(L, cd, L.ldL, split_stride, cd + 4 * comp_bytes, L.ldL, split_stride, rows32, L.ldP,
                                 L.ldP, 4, 1, at<double>(ws, L.M) + (size_t)sp * L.ldP * L.ldP, L.ldP, accumulate,
                                 ws, st)) != XTC_OK)
            return s;
    }
    return XTC_OK;
}

xtc_status split_rows_any(int form, const double* src, size_t n, void* dst, size_t split_stride, hipStream_t st) {
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 16384);
    if (form == 1) hipLaunchKernelGGL(k_split_rows<1>, dim3(blocks), dim3(256), 0, st, src, n, dst, split_stride);
    else if (form == 3) hipLaunchKernelGGL(k_split_rows<3>, dim3(blocks), dim3(256), 0, st, src, n, dst, split_stride);
    else hipLaunchKernelGGL(k_split_rows<6>, dim3(blocks), dim3(256), 0, st, src, n, dst, split_stride);
    return launched("split_rows");
}

// Split an FP64 row-major [nrows][ld] array into the k-packed operand format
// of k_nt_bf16 (split-BF16 forms).
xtc_status pack_kmajor_any(int form, const double* src, int nrows, int ld, void* dst, size_t split_stride,
                           hipStream_t st) {
    const size_t n = (size_t)nrows * (ld / 8);
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 16384);
    if (form == 3)
        hipLaunchKernelGGL(k_pack_kmajor<3>, dim3(blocks), dim3(256), 0, st, src, nrows, ld, (__bf16*)dst,
                           split_stride);
    else
        hipLaunchKernelGGL(k_pack_kmajor<6>, dim3(blocks), dim3(256), 0, st, src, nrows, ld, (__bf16*)dst,
                           split_stride);
    return launched("pack_kmajor");
}

// How an FP64 product of imax x jmax outputs over `rows` rows of ncomp
// components is laid out (k_gemm_tn_f64): the tile variant, the row segments
// and their length, by the time of its MFMAs (64 cycles each, one workgroup
// per CU and round) plus the sum over segments.  Large products take whole
// rows in 128 x 128 tiles; a product with fewer tiles than CUs is cut along
// the rows until the chip is full (N=8 on 2000 points is one tile: 1565 us in
// one piece), and the 64 x 64 tiles, whose waves share the rows, waste less on
// the padding of a small matrix.  A partial takes msize doubles; `bytes` are
// there for all of them.
struct TnF64Plan {
    int split, nseg, seg_rows;
};
TnF64Plan plan_tn_f64(int imax, int jmax, int ncomp, int rows, size_t msize, size_t bytes) {
    const size_t max_parts = std::min(bytes, kMpartF64Budget) / (msize * sizeof(double));
    TnF64Plan best{1, 1, (int)align_up((size_t)rows, 16)};
    double best_cycles = 1e300;
    for (int split = 1; split <= 4; split += 3) {
        const int tile = split == 1 ? 128 : 64;
        const long tiles = (long)((imax + tile - 1) / tile) * ((jmax + tile - 1) / tile);
        const int most = (int)std::min<size_t>({(size_t)kTnSplitMax, max_parts, (size_t)(rows + 31) / 32});
        for (int want = 1; want <= std::max(1, most); ++want) {
            const int seg = (int)align_up((size_t)((rows + want - 1) / want), 16);
            const int nseg = (rows + seg - 1) / seg;
            const double rounds = (double)((tiles * nseg + kCus - 1) / kCus);
            double c = rounds * (ncomp * (double)((seg + 4 * split - 1) / (4 * split)) * 1024.0 * (split == 1 ? 1.0 : 1.1) +
                                 (split == 1 ? 3000.0 : 6000.0));
            if (nseg > 1) c += 10000.0 + 1e-3 * 8.0 * nseg * (double)imax * jmax;   // about 2.4 TB/s at 2.4 GHz
            if (c < best_cycles) {
                best_cycles = c;
                best = {split, nseg, seg};
            }
        }
    }
    return best;
}

// M (+)= sum_c A_c^T B_c over `rows` rows in FP64 for outputs [0, imax) x
// [0, jmax) of M (leading dimension ldm, padded to whole 128 x 128 tiles).
xtc_status gemm_tn_f64(const Layout& L, const TnOperand& A, const TnOperand& B, int ncomp, int rows, int imax, int jmax,
                       double* M, int ldm, int accumulate, void* ws, hipStream_t st) {
    const size_t msize = align_up((size_t)imax, 128) * ldm;
    const TnF64Plan p = plan_tn_f64(imax, jmax, ncomp, rows, msize, scratch_bytes(L));
    const bool parts = p.nseg > 1;
    double* out = parts ? at<double>(ws, L.scr) : M;
    const int tile = p.split == 1 ? 128 : 64;
    const int n_it = (imax + tile - 1) / tile, n_jt = (jmax + tile - 1) / tile;
    const dim3 grid(n_it * n_jt, p.nseg);
    if (p.split == 1)
        hipLaunchKernelGGL(k_gemm_tn_f64<1>, grid, dim3(256), 0, st, A, B, ncomp, rows, n_it, p.seg_rows, out, ldm,
                           msize, parts ? 0 : accumulate);
    else
        hipLaunchKernelGGL(k_gemm_tn_f64<4>, grid, dim3(256), 0, st, A, B, ncomp, rows, n_it, p.seg_rows, out, ldm,
                           msize, parts ? 0 : accumulate);
    xtc_status s = launched("gemm_tn_f64");
    if (s != XTC_OK || !parts) return s;
    const int jmax4 = (int)align_up((size_t)jmax, 4);
    const size_t n4 = (size_t)imax * (jmax4 / 4);
    hipLaunchKernelGGL(k_reduce_M_f64, dim3((unsigned)std::min<size_t>((n4 + 255) / 256, 16384)), dim3(256), 0, st, out,
                       p.nseg, msize, ldm, imax, jmax4, M, accumulate);
    return launched("reduce_M_f64");
}

// One spin block of V2 from the accumulators, in slabs of rows P whose packed
// sums fit the scratch, or the one-body partials T1 and E (free at that time; at
// least kT1Split rows) if those hold more.
xtc_status finalize_V2(const Layout& L, const double* M1, const double* M2, double* V2, void* ws, hipStream_t st) {
    xtc_status s;
    const size_t t1e = L.e_end - L.T1;
    const bool big = scratch_bytes(L) > t1e;
    double* W = at<double>(ws, big ? L.scr : L.T1);
    const size_t bytes = big ? scratch_bytes(L) : t1e;
    const int slab = (int)std::min<size_t>(L.ldP, bytes / (L.ldP * sizeof(double)) / 32 * 32);
    for (int P0 = 0; P0 < L.Npair; P0 += slab) {
        const int np = std::min(slab, L.Npair - P0);
        hipLaunchKernelGGL(k_sym_sum, dim3(L.ldP / 32, (np + 31) / 32), dim3(256), 0, st, M1, M2, L.ldP, P0, W);
        if ((s = launched("sym_sum")) != XTC_OK) return s;
        hipLaunchKernelGGL(k_expand_V2, dim3((L.N + kExpandRows - 1) / kExpandRows, np), dim3(256), 0, st, W, L.ldP, P0,
                           L.N, V2);
        if ((s = launched("expand_V2")) != XTC_OK) return s;
    }
    return XTC_OK;
}

// The adjoint's X Gbar products in the split-BF16 3-product form (k_nt_bf16,
// FP32 accumulation over all pairs): Y_c (+)= X_c Gm^T for NC consecutive
// components sharing one right operand (X k-packed splits [NC][2][ldP/8][rows][8]
// with component stride a_comp, Gm k-packed splits [2][ldP/8][ldP][8], Y FP64
// [NC][cap][ldP] with component stride ystride).  The seven operands of a spin
// channel form two groups: D_{1..3} with Gbar, and rho, K^{x,y,z} with Gbar^T.
template <int NC>
xtc_status xg_group(const __bf16* X, size_t a_comp, size_t a_split, int rows, const __bf16* Gs, int ldP,
                    double* Y, size_t ystride, int accumulate, hipStream_t st) {
    const int n_rt = (rows + kLpRows - 1) / kLpRows, n_jt = (ldP + kPiThreads - 1) / kPiThreads;
    hipLaunchKernelGGL((k_nt_bf16<3, NC, false>), dim3(n_rt * n_jt), dim3(kPiThreads), 0, st, X, a_comp, a_split,
                       rows, Gs, (size_t)ldP * ldP, ldP, ldP, n_rt, (const d4*)nullptr, 0, 0, Y, ystride, ldP,
                       accumulate);
    return launched("gemm_xg_bf16");
}

// Row splits of the one-body term 1: kT1Split, more where few pairs leave the
// chip idle, if `bytes` hold their partials.
int t1_splits(const Layout& L, int rows, size_t bytes) {
    const int blocks = (L.Npair + 255) / 256;
    const int fit = (int)std::min<size_t>(kT1SplitMax, bytes / (L.ldP * sizeof(double)));
    return std::min(rows, std::max(kT1Split, std::min({kT1SplitMax, 1024 / blocks, fit})));
}

// Bytes beyond layout_bytes with which the launch plans of chunks of `rows` rows
// have the partials they ask for.  (None for the adjoint's workspaces: their
// own buffers leave the forward calls more than that.)
size_t plan_extra(Layout L, int rows) {
    if (L.bwd) return 0;
    const size_t all = (size_t)1 << 62;
    place_chunk(L, layout_bytes(L, align_up((size_t)rows, kRowQuant)), rows);
    const size_t have = L.end - (L.form != 0 ? L.kres : 0) - L.scr;
    size_t need = (size_t)t1_splits(L, rows, all) * L.ldP * sizeof(double);
    if (need <= (size_t)kT1Split * L.ldP * sizeof(double)) need = 0;
    if (L.form != 0) {
        const int nseg = (rows + L.segM - 1) / L.segM;
        need = std::max(need, std::min(nseg, m_seg_group(L, all)) * L.mslab);
    } else {
        const auto tn = [&](int imax, int ncomp) {
            const size_t msize = align_up((size_t)imax, 128) * L.ldP;
            const TnF64Plan p = plan_tn_f64(imax, L.Npair, ncomp, rows, msize, all);
            if (p.nseg > 1) need = std::max(need, p.nseg * msize * sizeof(double));
        };
        tn(L.Npair, 4);
        if (L.tc2) {
            tn(L.Npair, 1);
            tn(L.N * L.N, 3);
        }
    }
    return align_up(need > have ? need - have : 0, kAlign) + (L.form != 0 ? 0 : most_build_partials(L));
}

// The FP64 K build: in one piece, or split over g' where the grid is too small
// to fill the chip, the FP64 partials then summed into K.
xtc_status build_K_f64(const Layout& L, const JasDev& J, int g0, int rows, double* K, void* ws, hipStream_t st) {
    const KF64Plan p = plan_build_f64(L, rows, build_bytes(L));
    const bool parts = p.nseg > 1;
    double* out = parts ? at<double>(ws, L.kpart) : K;
    const hipError_t e = kf64_build(at<d4>(ws, L.pos), at<double>(ws, L.rho), L.ldP, L.ngp, g0, rows, J, p, out,
                                    parts ? p.ncol : L.ldP, st);
    if (e != hipSuccess) return fail(XTC_E_HIP, "build_K: %s", hipGetErrorString(e));
    if (!parts) return XTC_OK;
    const size_t n4 = (size_t)3 * rows * (L.ldP / 4);
    hipLaunchKernelGGL(k_reduce_K_f64, dim3((unsigned)std::min<size_t>((n4 + 255) / 256, 16384)), dim3(256), 0, st, out,
                       p.nseg, rows, p.ncol, L.ldP, K);
    return launched("reduce_K_f64");
}

xtc_status build_K_any(const Layout& L, const JasDev& J, int g0, int rows, double* K, int occ, void* ws,
                       hipStream_t st) {
    if (L.form != 0) return build_K_lp(L, g0, rows, J, K, occ, ws, st);
    return build_K_f64(L, J, g0, rows, K, ws, st);
}

}  // namespace

extern "C" {

int32_t xtc_pair_ld(int32_t N) { return N >= 1 ? pair_ld(N) : 0; }

const char* xtc_last_error(void) { return g_err.c_str(); }

size_t xtc_workspace_size(const xtc_problem* pb, int32_t prec, int32_t chunk_rows) {
    if (check_problem(pb) != XTC_OK) return 0;
    if (check_prec(prec) != XTC_OK) return 0;
    if (chunk_rows < 1 || chunk_rows > pb->Ng) {
        fail(XTC_E_ARG, "chunk_rows=%d outside [1,Ng]", chunk_rows);
        return 0;
    }
    const Layout L = make_layout(pb, prec);
    return layout_bytes(L, align_up((size_t)chunk_rows, kRowQuant)) + plan_extra(L, chunk_rows);
}

xtc_status xtc_prepare(const xtc_problem* pb, int32_t prec, int32_t chunk_rows, void* ws, size_t ws_bytes,
                       void* stream) {
    xtc_status s;
    if ((s = check_problem(pb)) != XTC_OK) return s;
    if ((s = check_prec(prec)) != XTC_OK) return s;
    Layout L = make_layout(pb, prec);
    L.cap = (int)chunk_capacity(L, ws_bytes);
    if ((s = check_ws(L, ws, ws_bytes)) != XTC_OK) return s;
    if (chunk_rows < 1 || chunk_rows > L.cap)
        return fail(XTC_E_WORKSPACE, "chunk_rows=%d exceeds the workspace capacity of %d rows", chunk_rows, L.cap);
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_prepare_pos, dim3((L.ngp + 255) / 256), dim3(256), 0, st, pb->xyz, L.Ng, L.ngp,
                       at<d4>(ws, L.pos));
    if ((s = launched("prepare_pos")) != XTC_OK) return s;
    const size_t lds = (size_t)L.N * kPrepRows * sizeof(double);
    hipLaunchKernelGGL(k_prepare_rho, dim3(L.ngp / kPrepRows), dim3(256), lds, st, pb->phi, pb->w, L.N, L.Ng,
                       L.ngp, L.ldP, at<double>(ws, L.rho));
    if ((s = launched("prepare_rho")) != XTC_OK) return s;
    if (L.form != 0) {
        if ((s = pack_any(L.form, at<double>(ws, L.rho), L.ngp, L.ldP, L.ldP, L.ngp / 8, L.ldL, at<void>(ws, L.rho_lp),
                          (size_t)L.ngp * L.ldL, st)) != XTC_OK)
            return s;
        hipLaunchKernelGGL(k_occ_pairs, dim3((L.ldO + 255) / 256), dim3(256), 0, st, make_occ(pb), L.N,
                           at<int>(ws, L.colmap), L.ldO);
        if ((s = launched("occ_pairs")) != XTC_OK) return s;
        hipLaunchKernelGGL(k_gather_occ, dim3(4096), dim3(256), 0, st, at<double>(ws, L.rho), L.ldP, L.ngp,
                           at<int>(ws, L.colmap), L.ldO, at<double>(ws, L.rho_occ));
        if ((s = launched("gather_occ")) != XTC_OK) return s;
        if (L.i8ok) {
            if ((s = fill(at<double>(ws, L.amax), (size_t)L.ldK8, st)) != XTC_OK) return s;
            if (occ_i8_prepare(at<double>(ws, L.rho_occ), L.ngp, L.ldO, L.nOP, L.i8,
                               at<unsigned long long>(ws, L.amax), at<void>(ws, L.stg), st) != hipSuccess)
                return fail(XTC_E_HIP, "occ_i8_prepare: %s", hipGetErrorString(hipGetLastError()));
        }
        // the adjoint's Pi operand: k-packed splits of rho (FP32: row-major)
        if (L.bwd && L.form == 1 &&
            (s = split_rows_any(L.form, at<double>(ws, L.rho), (size_t)L.ngp * L.ldP, at<void>(ws, L.rhoR),
                                (size_t)L.ngp * L.ldP, st)) != XTC_OK)
            return s;
        if (L.bwd && L.form != 1 &&
            (s = pack_kmajor_any(L.form, at<double>(ws, L.rho), L.ngp, L.ldP, at<void>(ws, L.rhoR),
                                 (size_t)L.ngp * L.ldP, st)) != XTC_OK)
            return s;
    }
    // zero the accumulators of every spin channel
    if ((s = fill(at<double>(ws, L.M), (size_t)L.nspin * L.ldP * L.ldP, st)) != XTC_OK) return s;
    if ((s = fill(at<double>(ws, L.h1acc), (size_t)L.nspin * L.ldP, st)) != XTC_OK) return s;
    if (L.tc2) {
        if ((s = fill(at<double>(ws, L.Atc), (size_t)L.ldP * L.ldP, st)) != XTC_OK) return s;
        if ((s = fill(at<double>(ws, L.Btc), (size_t)L.ldN * L.ldP, st)) != XTC_OK) return s;
    }
    return XTC_OK;
}

xtc_status xtc_build_K(const xtc_problem* pb, const xtc_jastrow* jas, int32_t g0, int32_t g1, int32_t prec,
                       double* K, void* ws, size_t ws_bytes, void* stream) {
    xtc_status s;
    JasDev J;
    if ((prec & XTC_K_REDUCED_OCC) && (prec & XTC_K_OCC_FP64))
        return fail(XTC_E_ARG, "prec: XTC_K_REDUCED_OCC and XTC_K_OCC_FP64 together");
    const int occ = (prec & XTC_K_REDUCED_OCC) ? kOccReduced : (prec & XTC_K_OCC_FP64) ? kOccFP64 : kOccExact;
    prec &= ~(XTC_K_REDUCED_OCC | XTC_K_OCC_FP64);
    if ((s = check_problem(pb)) != XTC_OK) return s;
    if ((s = check_prec(prec)) != XTC_OK) return s;
    if ((s = check_jastrow(jas, &J)) != XTC_OK) return s;
    if (!K) return fail(XTC_E_ARG, "K is NULL");
    if ((s = check_align(K, "K")) != XTC_OK) return s;
    Layout L = make_layout(pb, prec);
    place_chunk(L, ws_bytes, (long)g1 - g0);
    if ((s = check_ws(L, ws, ws_bytes)) != XTC_OK) return s;
    if ((s = check_range(L, g0, g1)) != XTC_OK) return s;
    return build_K_any(L, J, g0, g1 - g0, K, occ, ws, (hipStream_t)stream);
}

xtc_status xtc_contract_2body(const xtc_problem* pb, const double* K, int32_t g0, int32_t g1, int32_t prec,
                              int32_t flags, double* V2, void* ws, size_t ws_bytes, void* stream) {
    xtc_status s;
    if ((s = check_problem(pb)) != XTC_OK) return s;
    if ((s = check_prec(prec)) != XTC_OK) return s;
    if (!K) return fail(XTC_E_ARG, "K is NULL");
    if ((s = check_align(K, "K")) != XTC_OK) return s;
    if (flags & ~(XTC_RESET | XTC_FINALIZE)) return fail(XTC_E_ARG, "flags=%d unknown bits", flags);
    if ((flags & XTC_FINALIZE) && !V2) return fail(XTC_E_ARG, "V2 is NULL with XTC_FINALIZE");
    Layout L = make_layout(pb, prec);
    place_chunk(L, ws_bytes, (long)g1 - g0);
    if ((s = check_ws(L, ws, ws_bytes)) != XTC_OK) return s;
    if ((s = check_range(L, g0, g1)) != XTC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    if ((s = run_intermediates(L, pb, K, g0, g1, ws, st)) != XTC_OK) return s;
    const int rows = g1 - g0;
    if (L.form != 0) {
        if ((s = gemm2b_lp(L, K, g0, rows, (flags & XTC_RESET) ? 0 : 1, ws, st)) != XTC_OK) return s;
    } else {
        const double* rho_rows = at<double>(ws, L.rho) + (size_t)g0 * L.ldP;
        const size_t dstride = (size_t)L.crows * L.ldP;
        const TnOperand C{rho_rows, K, (size_t)rows * L.ldP, L.ldP};
        for (int sp = 0; sp < L.nspin; ++sp) {
            const double* D = at<double>(ws, L.D) + (size_t)sp * 4 * dstride;
            if ((s = gemm_tn_f64(L, C, TnOperand{D, D + dstride, dstride, L.ldP}, 4, rows, L.Npair, L.Npair,
                                 at<double>(ws, L.M) + (size_t)sp * L.ldP * L.ldP, L.ldP,
                                 (flags & XTC_RESET) ? 0 : 1, ws, st)) != XTC_OK)
                return s;
        }
    }
    if (flags & XTC_FINALIZE) {
        const size_t N4 = (size_t)L.N * L.N * L.N * L.N;
        const double* Ma = at<double>(ws, L.M);
        const double* Mb = Ma + (size_t)L.ldP * L.ldP;
        // closed shell: V2 = block (a, a); open shell: blocks (a, a), (a, b), (b, b)
        if ((s = finalize_V2(L, Ma, Ma, V2, ws, st)) != XTC_OK) return s;
        if (L.nspin == 2) {
            if ((s = finalize_V2(L, Ma, Mb, V2 + N4, ws, st)) != XTC_OK) return s;
            if ((s = finalize_V2(L, Mb, Mb, V2 + 2 * N4, ws, st)) != XTC_OK) return s;
        }
    }
    return XTC_OK;
}

xtc_status xtc_contract_1body_0body(const xtc_problem* pb, const double* K, int32_t g0, int32_t g1,
                                    int32_t prec, int32_t flags, double* h1, double* E0, void* ws,
                                    size_t ws_bytes, void* stream) {
    xtc_status s;
    if ((s = check_problem(pb)) != XTC_OK) return s;
    if ((s = check_prec(prec)) != XTC_OK) return s;
    if (!K) return fail(XTC_E_ARG, "K is NULL");
    if ((s = check_align(K, "K")) != XTC_OK) return s;
    if (flags & ~(XTC_RESET | XTC_FINALIZE | XTC_REUSE_INTERMEDIATES))
        return fail(XTC_E_ARG, "flags=%d unknown bits", flags);
    if ((flags & XTC_FINALIZE) && (!h1 || !E0)) return fail(XTC_E_ARG, "h1/E0 NULL with XTC_FINALIZE");
    Layout L = make_layout(pb, prec);
    place_chunk(L, ws_bytes, (long)g1 - g0);
    if ((s = check_ws(L, ws, ws_bytes)) != XTC_OK) return s;
    if ((s = check_range(L, g0, g1)) != XTC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    // the intermediates of this chunk (D = [A; B] and the per-row scalars S)
    // are in the workspace already when the two-body call has just made them
    if (!(flags & XTC_REUSE_INTERMEDIATES) && (s = run_intermediates(L, pb, K, g0, g1, ws, st)) != XTC_OK) return s;
    const int rows = g1 - g0;
    const double* rho_rows = at<double>(ws, L.rho) + (size_t)g0 * L.ldP;
    const size_t dstride = (size_t)L.crows * L.ldP;
    const int nsplit_t1 = t1_splits(L, rows, scratch_bytes(L));
    double* T1 = at<double>(ws, nsplit_t1 > kT1Split ? L.scr : L.T1);
    // exchange term: tiles of 64 outputs a side (16, 32 for smaller N), and row
    // splits until the four-wave workgroups fill the chip about twice
    const int tb = L.N <= 16 ? 1 : L.N <= 32 ? 2 : 4;
    const int n_t = (L.N + 16 * tb - 1) / (16 * tb);
    int nsplit_e = std::max(1, std::min(kESplitMax, 1024 / (n_t * n_t)));
    nsplit_e = std::min(nsplit_e, (rows + 7) / 8);
    const double* S = at<double>(ws, L.S);
    const size_t sstride = (size_t)L.crows * 8;
    // per spin channel (T1 and E are scratch of one channel at a time)
    for (int sp = 0; sp < L.nspin; ++sp) {
        const double* Ds = at<double>(ws, L.D) + (size_t)sp * 4 * dstride;
        hipLaunchKernelGGL(k_onebody_T1, dim3((L.Npair + 255) / 256, nsplit_t1), dim3(256), 0, st, rho_rows, K, Ds,
                           dstride, S + sp * sstride, L.nspin == 2 ? S + (1 - sp) * sstride : nullptr, rows, L.ldP,
                           L.Npair, T1);
        if ((s = launched("onebody_T1")) != XTC_OK) return s;
        const auto exchange = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(n_t * n_t, nsplit_e), dim3(256), 0, st, rho_rows, K, Ds, dstride, rows,
                               L.ldP, L.N, make_occ(pb, sp), at<double>(ws, L.E));
        };
        if (tb == 1) exchange(k_onebody_E<1>);
        else if (tb == 2) exchange(k_onebody_E<2>);
        else exchange(k_onebody_E<4>);
        if ((s = launched("onebody_E")) != XTC_OK) return s;
        hipLaunchKernelGGL(k_onebody_accumulate, dim3((L.Npair + 31) / 32), dim3(256), 0, st,
                           T1, nsplit_t1, at<double>(ws, L.E), nsplit_e, L.ldP, L.N,
                           at<double>(ws, L.h1acc) + (size_t)sp * L.ldP, (flags & XTC_RESET) ? 0 : 1);
        if ((s = launched("onebody_accumulate")) != XTC_OK) return s;
    }
    if (flags & XTC_FINALIZE) {
        const int NN = L.N * L.N;
        const double* ha = at<double>(ws, L.h1acc);
        hipLaunchKernelGGL(k_onebody_finalize, dim3((NN + 255) / 256), dim3(256), 0, st, ha,
                           L.nspin == 2 ? ha + L.ldP : nullptr, L.N, make_occ(pb, 0), make_occ(pb, 1), h1, E0);
        if ((s = launched("onebody_finalize")) != XTC_OK) return s;
    }
    return XTC_OK;
}

xtc_status xtc_backward(const xtc_problem* pb, const xtc_jastrow* jas, int32_t prec, const double* gV2,
                        const double* gh1, double gE0, double* gcoef, void* ws, size_t ws_bytes, void* stream) {
    xtc_status s;
    JasDev J;
    if ((s = check_problem(pb)) != XTC_OK) return s;
    if ((s = check_prec(prec)) != XTC_OK) return s;
    if ((s = check_jastrow(jas, &J)) != XTC_OK) return s;
    if (J.kind != 1) return fail(XTC_E_UNSUPPORTED, "the adjoint is taken with respect to power-form coefficients");
    if (!(prec & XTC_WITH_BACKWARD)) return fail(XTC_E_ARG, "prec must carry XTC_WITH_BACKWARD");
    if (!gcoef) return fail(XTC_E_ARG, "gcoef is NULL");
    if (!std::isfinite(gE0)) return fail(XTC_E_ARG, "gE0 not finite");
    Layout L = make_layout(pb, prec);
    place_chunk(L, ws_bytes, L.Ng);   // chunks of the capacity
    if ((s = check_ws(L, ws, ws_bytes)) != XTC_OK) return s;
    if (L.form == 0) {                // nothing of a chunk but Kc is live while its K is built
        L.kpart = L.S;
        L.kres = L.end - L.S;
    }
    hipStream_t st = (hipStream_t)stream;
    const bool open = L.nspin == 2;
    const OccList occ = make_occ(pb, 0);
    hipLaunchKernelGGL(k_occ_flags, dim3((L.N + 255) / 256), dim3(256), 0, st, occ, L.N, at<double>(ws, L.occw),
                       at<int>(ws, L.kidx));
    if ((s = launched("occ_flags")) != XTC_OK) return s;
    // adjoint of the packed accumulator(s): Gm[t] is the right operand of the
    // Cbar products (Gbar^t) and Gm[2 + t] that of the Abar, Bbar products
    // (Gbar^t transposed); closed shell: one symmetric Gbar for both
    const size_t gsz = (size_t)L.ldP * L.ldP;
    double* G = at<double>(ws, L.M);
    const double* Gm[4] = {G, G, G, G};
    if (!open) {
        hipLaunchKernelGGL(k_make_gbar, dim3((L.ldP + 255) / 256, L.ldP), dim3(256), 0, st, gV2, gh1, gE0,
                           at<double>(ws, L.occw), L.N, L.ldP, G);
    } else {
        double* GT = at<double>(ws, L.GT);
        hipLaunchKernelGGL(k_make_gbar_open, dim3((L.ldP + 255) / 256, L.ldP), dim3(256), 0, st, gV2, gh1, gE0,
                           at<double>(ws, L.occw), L.N, L.ldP, G, G + gsz, GT, GT + gsz);
        Gm[1] = G + gsz;
        Gm[2] = GT;
        Gm[3] = GT + gsz;
    }
    if ((s = launched("make_gbar")) != XTC_OK) return s;
    // the X Gbar products in split BF16 only in the 3-product form: the MFMA's
    // FP32 accumulation rounds with a small negative bias, which the six-product
    // form (twice the accumulations per k-step, and a smaller random error to
    // hide it) carries coherently into the gradient; it keeps them in FP64
    const bool bsplit = L.form == 3;
    const __bf16* Gs[4];
    for (int i = 0; i < 4; ++i) {
        const int slot = open ? i : 0;
        Gs[i] = at<__bf16>(ws, L.GsL) + (size_t)slot * L.ns * gsz;
        if (bsplit && (open || i == 0) &&
            (s = pack_kmajor_any(L.form, Gm[i], L.ldP, L.ldP, (void*)Gs[i], gsz, st)) != XTC_OK)
            return s;
    }
    const size_t ystride = (size_t)L.crows * L.ldP;
    double* Kc = at<double>(ws, L.Kc);
    double* Y = at<double>(ws, L.Y);
    const int n_jt_pi = L.ngp / 128;
    bool first = true;
    for (int g0 = 0; g0 < L.Ng; g0 += L.cap) {
        const int rows = std::min(L.cap, L.Ng - g0);
        const bool last = g0 + rows >= L.Ng;
        if ((s = build_K_any(L, J, g0, rows, Kc, kOccExact, ws, st)) != XTC_OK) return s;
        if ((s = run_intermediates(L, pb, Kc, g0, g0 + rows, ws, st)) != XTC_OK) return s;
        const double* rho_rows = at<double>(ws, L.rho) + (size_t)g0 * L.ldP;
        const size_t kstride = (size_t)rows * L.ldP;
        // Y slots: 0..2 Cbar_{1..3} = sum_t D^t_{1..3} Gbar^t^T, then per spin
        // channel t: 3 + 4t Abar^t = rho Gbar^t, 4 + 4t .. 6 + 4t Bbar^t = K Gbar^t
        const double* rk[4] = {rho_rows, Kc, Kc + kstride, Kc + 2 * kstride};
        const size_t a_split = (size_t)rows * L.ldP, a_comp = (size_t)L.ns * a_split;
        char* xs = at<char>(ws, L.KbL);
        // split-BF16: rho and K to k-packed splits once (slots 3..6), D^t (slots 0..2) per channel
        if (bsplit)
            for (int y = 0; y < 4; ++y)
                if ((s = pack_kmajor_any(L.form, rk[y], rows, L.ldP, xs + (3 + y) * a_comp * L.es, a_split, st)) !=
                    XTC_OK)
                    return s;
        for (int t = 0; t < L.nspin; ++t) {
            const double* D = at<double>(ws, L.D) + (size_t)t * 4 * ystride;
            const double* dsrc[3] = {D + ystride, D + 2 * ystride, D + 3 * ystride};
            double* Yab = Y + (size_t)(3 + 4 * t) * ystride;
            if (bsplit) {
                for (int y = 0; y < 3; ++y)
                    if ((s = pack_kmajor_any(L.form, dsrc[y], rows, L.ldP, xs + y * a_comp * L.es, a_split, st)) !=
                        XTC_OK)
                        return s;
                if ((s = xg_group<3>((const __bf16*)xs, a_comp, a_split, rows, Gs[t], L.ldP, Y, ystride, t, st)) !=
                    XTC_OK)
                    return s;
                if ((s = xg_group<4>((const __bf16*)(xs + 3 * a_comp * L.es), a_comp, a_split, rows, Gs[2 + t],
                                     L.ldP, Yab, ystride, 0, st)) != XTC_OK)
                    return s;
            } else {
                const int n_it = (rows + 63) / 64, n_jt = L.ldP / 128;
                XgProducts prod;
                for (int y = 0; y < kXgMax; ++y) {
                    prod.X[y] = y < 3 ? dsrc[y] : rk[y - 3];
                    prod.Y[y] = y < 3 ? Y + (size_t)y * ystride : Yab + (size_t)(y - 3) * ystride;
                    prod.G[y] = Gm[y < 3 ? t : 2 + t];
                    prod.accumulate[y] = y < 3 ? t : 0;
                }
                hipLaunchKernelGGL(k_gemm_xg_f64, dim3(n_it * n_jt, kXgMax), dim3(256), 0, st, prod, rows, L.ldP,
                                   (int)align_up((size_t)L.Npair, 16), n_jt);
                if ((s = launched("gemm_xg")) != XTC_OK) return s;
            }
        }
        const size_t lds = (size_t)L.nocc * L.N * 4 * sizeof(double);
        if (lds > 64 * 1024) {
            const hipError_t e = hipFuncSetAttribute((const void*)k_adj_T, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)lds);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                return fail(XTC_E_HIP, "adj_T LDS attribute: %s", hipGetErrorString(e));
            }
        }
        for (int t = 0; t < L.nspin; ++t) {
            hipLaunchKernelGGL(k_adj_T, dim3(std::min(rows, 16384)), dim3(64 * std::min(4, (L.N + 15) / 16)), lds, st, rho_rows, Kc,
                               Y + (size_t)4 * t * ystride, ystride, rows, L.ldP, L.N, make_occ(pb, t),
                               at<double>(ws, L.T), at<double>(ws, L.Wbar), t);
            if ((s = launched("adj_T")) != XTC_OK) return s;
        }
        const size_t nel = (size_t)rows * L.Npair;
        hipLaunchKernelGGL(k_adj_assemble, dim3((unsigned)std::min<size_t>((nel + 255) / 256, 16384)), dim3(256), 0, st,
                           Y, ystride, at<double>(ws, L.S), at<double>(ws, L.T), at<double>(ws, L.Wbar),
                           at<int>(ws, L.kidx), at<double>(ws, L.occw), rows, L.ldP, L.N, L.nocc, L.nspin);
        if ((s = launched("adj_assemble")) != XTC_OK) return s;
        const int n_it_pi = (rows + 31) / 32;
        int nblk_pi;
        if (L.form == 0) {
            nblk_pi = n_it_pi * n_jt_pi;
            hipLaunchKernelGGL(k_pi_grad, dim3(nblk_pi), dim3(256), 0, st, Y, ystride, rows, at<double>(ws, L.rho),
                               L.ldP, (int)align_up((size_t)L.Npair, 16), at<d4>(ws, L.pos), g0, L.ngp, n_jt_pi, J.ncoef, at<double>(ws, L.gpart));
            if ((s = launched("pi_grad")) != XTC_OK) return s;
        } else {
            // Kbar of the chunk to split operands (FP32: row-major; split BF16:
            // k-packed), then the reduced Pi tiles
            const size_t kb_split = (size_t)rows * L.ldP, kb_comp = (size_t)L.ns * kb_split;
            char* kb = at<char>(ws, L.KbL);
            for (int x = 0; x < 3; ++x) {
                s = L.form == 1 ? split_rows_any(L.form, Y + x * ystride, (size_t)rows * L.ldP,
                                                 kb + x * kb_comp * L.es, kb_split, st)
                                : pack_kmajor_any(L.form, Y + x * ystride, rows, L.ldP, kb + x * kb_comp * L.es,
                                                  kb_split, st);
                if (s != XTC_OK) return s;
            }
            const size_t rr_split = (size_t)L.ngp * L.ldP;
            if (L.form == 1) {
                const int n_jt_lp = (L.ngp + 255) / 256;
                nblk_pi = n_it_pi * n_jt_lp;
                hipLaunchKernelGGL(k_pi_grad_lp<1>, dim3(nblk_pi), dim3(256), 0, st, (const void*)kb, kb_comp, kb_split,
                                   rows, at<void>(ws, L.rhoR), rr_split, L.ldP, at<d4>(ws, L.pos), g0, L.ngp, n_jt_lp,
                                   J.ncoef, at<double>(ws, L.gpart));
            } else {
                const int n_rt = (rows + kLpRows - 1) / kLpRows;
                const int n_jt = (L.ngp + kPiThreads - 1) / kPiThreads;
                nblk_pi = n_rt * n_jt;
                const __bf16* kbb = (const __bf16*)kb;
                const __bf16* rrb = at<__bf16>(ws, L.rhoR);
                if (L.form == 3)
                    hipLaunchKernelGGL((k_nt_bf16<3, 3, true>), dim3(nblk_pi), dim3(kPiThreads), 0, st, kbb, kb_comp,
                                       kb_split, rows, rrb, rr_split, L.ngp, L.ldP, n_rt, at<d4>(ws, L.pos), g0,
                                       J.ncoef, at<double>(ws, L.gpart), (size_t)0, 0, 0);
                else
                    hipLaunchKernelGGL((k_nt_bf16<6, 3, true>), dim3(nblk_pi), dim3(kPiThreads), 0, st, kbb, kb_comp,
                                       kb_split, rows, rrb, rr_split, L.ngp, L.ldP, n_rt, at<d4>(ws, L.pos), g0,
                                       J.ncoef, at<double>(ws, L.gpart), (size_t)0, 0, 0);
            }
            if ((s = launched("pi_grad_lp")) != XTC_OK) return s;
        }
        hipLaunchKernelGGL(k_reduce_grad, dim3(J.ncoef), dim3(256), 0, st, at<double>(ws, L.gpart), nblk_pi, J.ncoef,
                           at<double>(ws, L.gacc), first ? 0 : 1, last ? gcoef : nullptr);
        if ((s = launched("reduce_grad")) != XTC_OK) return s;
        first = false;
    }
    return XTC_OK;
}

// ------------------------------------------------------------- Loewdin --
namespace {
constexpr int kLowdinSeg = 4096;
constexpr int kJacobiMaxSweeps = 40;
// Bytes of S partials that shorter segments than kLowdinSeg may take.
constexpr size_t kLowdinPartBudget = (size_t)32 << 20;
struct LowdinLayout {
    int ldS, nseg, seg;
    int pass_sweeps;     // Jacobi sweeps whose rotations fit where the partials were
    size_t part, S, U, X, rot, sweeps, status, total;
};
// full: segments short enough that the tiles of a mid-size grid fill the chip,
// with partials of at most kLowdinPartBudget (or those of kLowdinSeg points each),
// and room for the rotations of every sweep the eigensolver may take.  Otherwise
// segments of kLowdinSeg points, and as many sweeps at a time as their partials
// leave room for (at least one: 8 N' (N' - 1) bytes, N' = N rounded up to even).
LowdinLayout lowdin_layout(int N, int Ng, bool full) {
    LowdinLayout L{};
    L.ldS = (int)align_up((size_t)N, 64);
    const size_t psize = (size_t)L.ldS * L.ldS * sizeof(double);
    const int want = (int)std::min<size_t>(256, kLowdinPartBudget / psize);
    L.seg = !full || Ng <= 128 ? kLowdinSeg
                               : std::min(kLowdinSeg, std::max(64, (int)align_up((size_t)((Ng + want - 1) / want), 16)));
    L.nseg = (Ng + L.seg - 1) / L.seg;
    const size_t Np = align_up((size_t)N, 2), sweep = (Np - 1) * (Np / 2) * 2 * sizeof(double);
    size_t off = 0;
    L.part = L.rot = off;
    off = align_up(off + std::max(L.nseg * psize, full ? kJacobiMaxSweeps * sweep : 0), kAlign);
    L.pass_sweeps = (int)std::min<size_t>(kJacobiMaxSweeps, off / sweep);
    L.S = off;      off = align_up(off + (size_t)N * N * sizeof(double), kAlign);
    L.U = off;      off = align_up(off + (size_t)N * N * sizeof(double), kAlign);
    L.X = off;      off = align_up(off + (size_t)N * N * sizeof(double), kAlign);
    L.sweeps = off; off = align_up(off + 2 * sizeof(int), kAlign);
    L.status = off; off = align_up(off + 2 * sizeof(double), kAlign);
    L.total = off;
    return L;
}
// The full layout if `bytes` hold it, else the small one.
LowdinLayout lowdin_layout_for(int N, int Ng, size_t bytes) {
    const LowdinLayout L = lowdin_layout(N, Ng, true);
    return L.total <= bytes ? L : lowdin_layout(N, Ng, false);
}

xtc_status check_lowdin_args(int N, int Ng, const double* chi, const double* w, const double* phi) {
    if (N < 1 || N > kMaxN || Ng < 1) return fail(XTC_E_ARG, "N=%d or Ng=%d out of range", N, Ng);
    if (Ng > kMaxNg) return fail(XTC_E_UNSUPPORTED, "Ng=%d above %d", Ng, kMaxNg);
    if (!chi || !w || !phi) return fail(XTC_E_ARG, "NULL array");
    return XTC_OK;
}

xtc_status run_lowdin(const LowdinLayout& L, int N, int Ng, const double* chi, const double* w, double* phi,
                      double* lambda, void* ws, hipStream_t st);

// Scratch of xtc_lowdin_noalloc: a file-scope device array, one copy per
// device the library runs on (held until the process ends).  In host code
// `scratch` names the symbol only; its device address on each device comes
// from hipGetSymbolAddress, taken once per device with that device current.
constexpr size_t kNoAllocBytes = XTC_LOWDIN_NOALLOC_BYTES;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

static __device__ __align__(256) unsigned char scratch[XTC_LOWDIN_NOALLOC_BYTES];

namespace {
xtc_status scratch_of_current_device(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(XTC_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    }
    if (dev < 0 || dev >= kMaxDevices) return fail(XTC_E_UNSUPPORTED, "device %d above %d", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return fail(XTC_E_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return XTC_OK;
}
}  // namespace

xtc_status xtc_tc_2body(const xtc_problem* pb, const xtc_jastrow* jas, const double* dphi, const double* K,
                        int32_t g0, int32_t g1, int32_t prec, int32_t flags, double* K2, void* ws, size_t ws_bytes,
                        void* stream) {
    xtc_status s;
    JasDev J;
    if ((s = check_problem(pb)) != XTC_OK) return s;
    if ((s = check_prec(prec)) != XTC_OK) return s;
    if ((s = check_jastrow(jas, &J)) != XTC_OK) return s;
    if (!(prec & XTC_WITH_TC2)) return fail(XTC_E_ARG, "prec must carry XTC_WITH_TC2");
    if (!dphi || !K) return fail(XTC_E_ARG, "dphi or K is NULL");
    if ((s = check_align(K, "K")) != XTC_OK) return s;
    if (flags & ~(XTC_RESET | XTC_FINALIZE)) return fail(XTC_E_ARG, "flags=%d unknown bits", flags);
    if ((flags & XTC_FINALIZE) && !K2) return fail(XTC_E_ARG, "K2 is NULL with XTC_FINALIZE");
    Layout L = make_layout(pb, prec);
    place_chunk(L, ws_bytes, (long)g1 - g0);
    if ((s = check_ws(L, ws, ws_bytes)) != XTC_OK) return s;
    if ((s = check_range(L, g0, g1)) != XTC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    const int rows = g1 - g0;
    // F for the chunk rows: scalar kernel S against all g', in the arithmetic of
    // prec (reduced forms: the K-build kernel with one component, segment
    // partials in the K-build partial buffer, FP64 reduction)
    double* F = at<double>(ws, L.Ftc);
    if (L.form == 0) {
        const int n_rt = (rows + kKRows - 1) / kKRows;
        const dim3 gF(n_rt * (L.ldP / 128));
        if (J.kind == 0)
            hipLaunchKernelGGL((k_build_F_f64<0, 8>), gF, dim3(256), 0, st, at<d4>(ws, L.pos), at<double>(ws, L.rho),
                               L.ldP, L.ngp, g0, rows, n_rt, J, F);
        else
            hipLaunchKernelGGL((k_build_F_f64<1, 8>), gF, dim3(256), 0, st, at<d4>(ws, L.pos), at<double>(ws, L.rho),
                               L.ldP, L.ngp, g0, rows, n_rt, J, F);
    } else if ((s = build_lp_pieces<1>(L, g0, rows, J, F, ws, st)) != XTC_OK) {
        return s;
    }
    if ((s = launched("build_F")) != XTC_OK) return s;
    const int acc = (flags & XTC_RESET) ? 0 : 1;
    const double* rho_rows = at<double>(ws, L.rho) + (size_t)g0 * L.ldP;
    double* Atc = at<double>(ws, L.Atc);
    double* Btc = at<double>(ws, L.Btc);
    if (L.form == 0) {
        double* Rg = at<double>(ws, L.Rg);
        const size_t xs = (size_t)L.crows * L.ldN;
        const size_t nrg = (size_t)rows * L.ldN;
        hipLaunchKernelGGL(k_rhog, dim3((unsigned)std::min<size_t>((nrg + 255) / 256, 16384)), dim3(256), 0, st, pb->w,
                           pb->phi, dphi, L.N, L.Ng, g0, rows, L.ldN, xs, Rg);
        if ((s = launched("rhog")) != XTC_OK) return s;
        if ((s = gemm_tn_f64(L, TnOperand{rho_rows, rho_rows, 0, L.ldP}, TnOperand{F, F, 0, L.ldP}, 1, rows, L.Npair,
                             L.Npair, Atc, L.ldP, acc, ws, st)) != XTC_OK)
            return s;
        const size_t ks = (size_t)rows * L.ldP;
        if ((s = gemm_tn_f64(L, TnOperand{Rg, Rg + xs, xs, L.ldN}, TnOperand{K, K + ks, ks, L.ldP}, 3, rows, L.N * L.N,
                             L.Npair, Btc, L.ldP, acc, ws, st)) != XTC_OK)
            return s;
    } else {
        // reduced forms: both contractions as split products over the chunk rows,
        // FP32 partials per segM rows, FP64 reduction into the accumulators
        const int rows32 = (int)align_up((size_t)rows, kRowQuant);
        const int n8 = rows32 / 8;
        char* cd = at<char>(ws, L.CDlp);
        const size_t sL = (size_t)L.crows * L.ldL, sN = (size_t)L.crows * L.ldN;   // elements of one split
        const size_t cL = (size_t)L.ns * sL * L.es, cN = (size_t)L.ns * sN * L.es;   // bytes of one component
        if ((s = pack_any(L.form, rho_rows, rows, L.ldP, L.ldP, n8, L.ldL, cd, sL, st)) != XTC_OK) return s;
        if ((s = pack_any(L.form, F, rows, L.ldP, L.ldP, n8, L.ldL, cd + cL, sL, st)) != XTC_OK) return s;
        if ((s = gemm_tn_grouped(L, cd, L.ldL, sL, cd + cL, L.ldL, sL, rows32, L.ldP, L.ldP, 1, 1, Atc, L.ldP, acc, ws,
                                 st)) != XTC_OK)
            return s;
        char* kd = cd + 3 * cN;
        const size_t ks = (size_t)rows * L.ldP;
        const auto rhog = L.form == 1 ? k_pack_rhog<1> : L.form == 3 ? k_pack_rhog<3> : k_pack_rhog<6>;
        hipLaunchKernelGGL(rhog, dim3((L.ldN + 255) / 256, n8, 3), dim3(256), 0, st, pb->w, pb->phi, dphi, L.N, L.Ng, g0,
                           rows, L.ldN, cd, sN, L.ns * sN);
        if ((s = launched("pack_rhog")) != XTC_OK ||
            (s = pack_many(L.form, PackSrc{{K, K + ks, K + 2 * ks}}, 3, rows, L.ldP, L.ldP, n8, L.ldL, kd, sL,
                           L.ns * sL, st)) != XTC_OK)
            return s;
        // the three components of rhog_pq . K_R summed inside each workgroup
        if ((s = gemm_tn_grouped(L, cd, L.ldN, sN, kd, L.ldL, sL, rows32, L.N * L.N, L.ldP, 3, 3, Btc, L.ldP, acc, ws,
                                 st)) != XTC_OK)
            return s;
    }
    if (flags & XTC_FINALIZE) {
        const int NN = L.N * L.N;
        hipLaunchKernelGGL(k_finalize_K2, dim3((NN + 255) / 256, L.N, L.N), dim3(256), 0, st, Atc, L.ldP, Btc, L.N,
                           K2);
        if ((s = launched("finalize_K2")) != XTC_OK) return s;
    }
    return XTC_OK;
}

xtc_status xtc_frozen_core(int32_t N, const double* V2, const double* h1, const double* E0, int32_t ncore,
                           const int32_t* core, int32_t nact, const int32_t* act, double* V2_act, double* h1_act,
                           double* E_fc, void* stream) {
    if (N < 1 || N > kMaxN) return fail(XTC_E_ARG, "N=%d outside [1,%d]", N, kMaxN);
    if (ncore < 0 || ncore > kMaxFcList || nact < 1 || nact > kMaxFcList || ncore + nact > N)
        return fail(XTC_E_ARG, "ncore=%d, nact=%d invalid for N=%d", ncore, nact, N);
    if (!V2 || !h1 || !E0 || !act || (ncore > 0 && !core) || !V2_act || !h1_act || !E_fc)
        return fail(XTC_E_ARG, "NULL argument");
    std::vector<char> seen(N, 0);
    IdxList c{}, a{};
    c.n = ncore;
    a.n = nact;
    for (int i = 0; i < ncore + nact; ++i) {
        const int k = i < ncore ? core[i] : act[i - ncore];
        if (k < 0 || k >= N) return fail(XTC_E_ARG, "orbital %d outside [0,N)", k);
        if (seen[k]) return fail(XTC_E_ARG, "orbital %d listed twice (core and active must be disjoint)", k);
        seen[k] = 1;
        if (i < ncore) c.k[i] = k;
        else a.k[i - ncore] = k;
    }
    hipStream_t st = (hipStream_t)stream;
    const int n_h = (nact * nact + 255) / 256;
    hipLaunchKernelGGL(k_frozen_core, dim3(1 + n_h + nact * nact), dim3(256), 0, st, V2, h1, E0, N, c, a, n_h, V2_act,
                       h1_act, E_fc);
    return launched("frozen_core");
}

size_t xtc_lowdin_workspace_size(int32_t N, int32_t Ng) {
    if (N < 1 || N > kMaxN || Ng < 1 || Ng > kMaxNg) {
        fail(Ng > kMaxNg ? XTC_E_UNSUPPORTED : XTC_E_ARG, "N=%d or Ng=%d out of range", N, Ng);
        return 0;
    }
    return lowdin_layout(N, Ng, true).total;
}

xtc_status xtc_lowdin(int32_t N, int32_t Ng, const double* chi, const double* w, double* phi, double* lambda,
                      void* ws, size_t ws_bytes, void* stream) {
    xtc_status s;
    if ((s = check_lowdin_args(N, Ng, chi, w, phi)) != XTC_OK) return s;
    if (!ws) return fail(XTC_E_WORKSPACE, "workspace is NULL");
    if ((uintptr_t)ws % kAlign) return fail(XTC_E_WORKSPACE, "workspace not 256-byte aligned");
    const LowdinLayout L = lowdin_layout_for(N, Ng, ws_bytes);
    if (ws_bytes < L.total) return fail(XTC_E_WORKSPACE, "workspace of %zu bytes < %zu", ws_bytes, L.total);
    return run_lowdin(L, N, Ng, chi, w, phi, lambda, ws, (hipStream_t)stream);
}

xtc_status xtc_lowdin_noalloc(int32_t N, int32_t Ng, const double* chi, const double* w, double* phi,
                              double* lambda, void* stream) {
    xtc_status s;
    if ((s = check_lowdin_args(N, Ng, chi, w, phi)) != XTC_OK) return s;
    const LowdinLayout L = lowdin_layout_for(N, Ng, kNoAllocBytes);
    if (L.total > kNoAllocBytes)
        return fail(XTC_E_UNSUPPORTED, "N=%d, Ng=%d needs %zu bytes of scratch, above the %zu of the static array", N,
                    Ng, L.total, kNoAllocBytes);
    void* ws = nullptr;
    if ((s = scratch_of_current_device(&ws)) != XTC_OK) return s;
    return run_lowdin(L, N, Ng, chi, w, phi, lambda, ws, (hipStream_t)stream);
}
}  // extern "C"

namespace {
xtc_status run_lowdin(const LowdinLayout& L, int N, int Ng, const double* chi, const double* w, double* phi,
                      double* lambda, void* ws, hipStream_t st) {
    xtc_status s;
    const int n_t = L.ldS / 64;
    hipLaunchKernelGGL(k_syrk_w_part, dim3(n_t * (n_t + 1) / 2, L.nseg), dim3(256), 0, st, chi, w, N, Ng, L.ldS, n_t,
                       L.seg, at<double>(ws, L.part));
    if ((s = launched("syrk_w")) != XTC_OK) return s;
    const int NN = N * N;
    hipLaunchKernelGGL(k_syrk_reduce, dim3((NN + 255) / 256), dim3(256), 0, st, at<double>(ws, L.part), L.nseg, N,
                       L.ldS, at<double>(ws, L.S));
    if ((s = launched("syrk_reduce")) != XTC_OK) return s;
    const size_t lds = N <= kJacobiLdsN ? (size_t)N * N * sizeof(double) : 0;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_jacobi<true>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(XTC_E_HIP, "jacobi LDS attribute: %s", hipGetErrorString(e));
        }
    }
    // (a pass on a matrix that has converged changes nothing)
    for (int done = 0; done < kJacobiMaxSweeps; done += L.pass_sweeps) {
        hipLaunchKernelGGL((lds ? k_jacobi<true> : k_jacobi<false>), dim3(1), dim3(kJacobiThreads), lds, st,
                           at<double>(ws, L.S), N, std::min(L.pass_sweeps, kJacobiMaxSweeps - done), done > 0 ? 1 : 0,
                           at<double>(ws, L.rot), at<int>(ws, L.sweeps));
        if ((s = launched("jacobi")) != XTC_OK) return s;
        hipLaunchKernelGGL(k_jacobi_vectors, dim3(N), dim3(64), 0, st, at<double>(ws, L.rot), at<int>(ws, L.sweeps), N,
                           done > 0 ? 1 : 0, at<double>(ws, L.U));
        if ((s = launched("jacobi_vectors")) != XTC_OK) return s;
    }
    // convergence and positive definiteness are checked before anything is
    // written to phi or lambda (one synchronisation of the stream)
    hipLaunchKernelGGL(k_lowdin_status, dim3(1), dim3(64), 0, st, at<double>(ws, L.S), N, at<int>(ws, L.sweeps),
                       at<double>(ws, L.status));
    if ((s = launched("lowdin_status")) != XTC_OK) return s;
    double stat[2] = {0.0, 0.0};
    hipError_t e = hipMemcpyAsync(stat, at<double>(ws, L.status), sizeof stat, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(XTC_E_HIP, "lowdin status read-back: %s", hipGetErrorString(e));
    if (stat[0] >= kJacobiMaxSweeps)
        return fail(XTC_E_ARG, "Jacobi eigensolver of the grid overlap did not converge in %d sweeps",
                    kJacobiMaxSweeps);
    if (!(stat[1] > 0.0))
        return fail(XTC_E_ARG, "grid overlap matrix is not positive definite (smallest eigenvalue %g)", stat[1]);
    hipLaunchKernelGGL(k_inv_sqrt, dim3((NN + 255) / 256), dim3(256), 0, st, at<double>(ws, L.S), at<double>(ws, L.U),
                       N, at<double>(ws, L.X));
    if ((s = launched("inv_sqrt")) != XTC_OK) return s;
    const size_t xlds = align_up((size_t)N, 4) * 64 * sizeof(double);
    if (xlds > 64 * 1024) {
        e = hipFuncSetAttribute((const void*)k_apply_X, hipFuncAttributeMaxDynamicSharedMemorySize, (int)xlds);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(XTC_E_HIP, "apply_X LDS attribute: %s", hipGetErrorString(e));
        }
    }
    hipLaunchKernelGGL(k_apply_X, dim3((Ng + kApplyPoints - 1) / kApplyPoints, (N + 63) / 64), dim3(256), xlds, st,
                       at<double>(ws, L.X), chi, N, Ng, phi);
    if ((s = launched("apply_X")) != XTC_OK) return s;
    if (lambda) {
        hipLaunchKernelGGL(k_diag_copy, dim3((N + 255) / 256), dim3(256), 0, st, at<double>(ws, L.S), N, lambda);
        if ((s = launched("diag_copy")) != XTC_OK) return s;
    }
    return XTC_OK;
}
}  // namespace
