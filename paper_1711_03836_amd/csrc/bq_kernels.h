// Host-side launch interface of the HIP kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "bq_device.h"

namespace bq {

// Epilogues fused into the hopping kernel.  `hop` is D (or D^dag) applied to
// the input field at the output site, `v` a field on the output parity.
enum {
    EPI_HOP = 0,   // out = a*v + f*hop                     (D_eo, D_oe, source preparation)
    EPI_TINV = 1,  // out = C (a*v + f*hop), C = clover blocks given (T_ee^-1 for K1 / reconstruction)
    EPI_TV = 2,    // out = C v + f*hop (+ |out|^2 partials)  (K2 of Mhat, full M)
    EPI_TVR = 3,   // w = C v + f*hop; r_out = r_in - alpha*w (+ |r_out|^2 partials)  (CG residual update)
};

// most columns one launch can give their own operator (kappa, clover)
constexpr int kMaxCols = 32;

struct FieldArg {
    void* d = nullptr;       // storage units
    float* s = nullptr;      // FP16 per-site scales
    size_t cstride = 0;      // units between columns
    size_t sstride = 0;      // floats between scale columns
};

struct HopLaunch {
    int prec = PREC_F64;     // storage precision of in/out/v/links/clover
    int rprec = PREC_F64;    // precision of r_in/r_out (EPI_TVR)
    int recon = 18;          // 18 or 12 reals per link
    int dagger = 0;
    int epi = EPI_HOP;
    int R = 1;               // columns per thread
    int bs = 256;            // sites per workgroup (a multiple of 64)
    int march = 0;           // > 0: t-marching kernel with segments of `march` time planes
                             //      (needs whole tiles per (x,y) plane and march | L_t)
    int lds = 0;             // 1: tile-shared kernel (links and clover staged in LDS) when a tile has
                             //    several column groups; 2: the same with one column per wave and the
                             //    x and y neighbour spinors exchanged between lanes
    int split = 0;           // 1: hop-split kernel, one workgroup per tile and column (R = 1; march and lds ignored)
    int last_t = 0;          // 1: the tiles are walked down in t, slice by slice (the +t neighbour's last read)
    Geom g{};
    int parity = 0;          // output parity
    int ncol = 1;
    const void* U[8] = {};   // links [parity*4 + mu], each on its own parity
    FieldArg in, out, v, r_in, r_out;
    const void* clov = nullptr;   // clover blocks on the output parity
    const double* alpha = nullptr;
    double* partial = nullptr;    // |.|^2 per wavefront of 64 sites: partial[c * pstride + wave]
    int nwaves = 0;               // waves of this launch (bound on `wave`)
    int pstride = 0;              // partial entries per column
    const int* status = nullptr;
    int statmask = 1;
    double ef = 1, eb = 1;   // time-hop coefficients of the forward / backward term
    int tbc = -1;
    double f = 1, a = 0;
    int percol = 0;                    // 1: column c uses cclov[c] and cf[c] instead of clov and f
    const void* cclov[kMaxCols] = {};
    double cf[kMaxCols] = {};
    // EPI_TVR, up to kFusedParts partials: alpha = cg_rho / (the sum of column c's nwaves partials at pap + c * pstride) is
    // taken by the kernel itself (0 if that sum is not positive and finite), which also writes alpha and pAp
    const double* pap = nullptr;
    const double* cg_rho = nullptr;
    double* cg_alpha = nullptr;
    double* cg_pAp = nullptr;
};

hipError_t launch_hop(const HopLaunch& L, hipStream_t st);
bool hop_variant_exists(int prec, int rprec, int recon, int R, int epi);

// clover
// B = sum_{mu<nu} sigma (x) F per parity (independent of kappa and c_SW) from the FP64 18-real links
hipError_t launch_clover_build(const Geom& g, const double2* const U64[8], double2* const B[2], hipStream_t st);
// T = 1 + ck*B and T^-1 of one parity, packed, in each storage precision whose pointer is not null;
// bad is set to 1 if a block is not positive definite (checked where an inverse is asked for)
hipError_t launch_clover_from_B(const Geom& g, const double2* B, double ck, void* const T[3], void* const Tinv[3],
                                int* bad, hipStream_t st);
hipError_t launch_clover_apply(int prec, const Geom& g, const void* clov, FieldArg in, FieldArg out, int ncol,
                               hipStream_t st, const void* const* cclov = nullptr, const int* status = nullptr,
                               int statmask = 0);

// layout conversion
// canonical links into the 18-real forms ([parity*4 + mu]); partial: links_take_parts maxima of the
// links' distance from SU(3)
int links_take_parts(const Geom& g);
hipError_t launch_links_take(const double2* canon, const Geom& g, const void* const d18[8], const void* const f18[8],
                             double* partial, hipStream_t st);
// the two-row forms from the FP64 18-real one; entries of a form that is not kept are null
hipError_t launch_links_rows(const void* const d18[8], int Vh, const void* const d12[8], const void* const f12[8],
                             const void* const h12[8], hipStream_t st);
// np parities from p0 on at once; dst / src: the field of parity p0, half_units (half_sites: scales) to the next
hipError_t launch_spinor_import(const double2* canon, int ncol, const Geom& g, int p0, int np, int prec, FieldArg dst,
                                size_t half_units, size_t half_sites, hipStream_t st);
hipError_t launch_spinor_export(FieldArg src, int ncol, const Geom& g, int p0, int np, int prec, size_t half_units,
                                size_t half_sites, double2* canon, hipStream_t st);
hipError_t launch_plaquette(const Geom& g, const double2* const U64[8], double* partial, int nparts, hipStream_t st);

// BLAS-1 and reductions
hipError_t launch_convert(int src_prec, FieldArg src, int dst_prec, FieldArg dst, int Vh, int ncol,
                          const int* status, int statmask, hipStream_t st);
hipError_t launch_norm2(int prec, FieldArg x, int Vh, int ncol, double* partial, int nwaves, hipStream_t st);
hipError_t launch_zero(int prec, FieldArg x, int Vh, int ncol, const int* status, int statmask, hipStream_t st);
hipError_t launch_copy16(const void* src, void* dst, size_t n16, hipStream_t st);  // n16 16-byte words
// x += alpha p ; p = r + beta p   (CG; per column, by status)
hipError_t launch_cg_update(int xprec, FieldArg x, int pprec, FieldArg p, int rprec, FieldArg r, int Vh, int ncol,
                            const double* alpha, const double* beta, const int* status, hipStream_t st);
// reliable update pieces: y += x (x low precision), x = 0
hipError_t launch_accum(int xprec, FieldArg x, FieldArg y64, int Vh, int ncol, const int* status, int statmask,
                        hipStream_t st);
// p = lowp(r64) + beta p (restart after a reliable update), rs = lowp(r64)
hipError_t launch_restart(FieldArg r64, int rsprec, FieldArg rs, int pprec, FieldArg p, int Vh, int ncol,
                          const double* beta, const int* flag, hipStream_t st);
// <x, y> (gamma5: <x, gamma_5 y>) per column, FP64; partials [col][re/im][wave]
hipError_t launch_dot(int prec, FieldArg x, FieldArg y, int Vh, int ncol, double* partial, int nwaves,
                      hipStream_t st, int gamma5 = 0);
hipError_t launch_z2_noise(uint64_t seed, long n0, const Geom& g, int parity, FieldArg dst, int ncol,
                           hipStream_t st);

// y += a x per column (a real, the same for every column) with |y|^2 partials per wave (FP64)
hipError_t launch_axpy_norm(FieldArg x, FieldArg y, double a, int n, int ncol, double* partial, int nwaves,
                            hipStream_t st);

// ---------------------------------------------------------------------------
// multishift CG: (A + sigma_k) x_k = b for all shifts in the Krylov space of the base system
// A + sigma_b (sigma_b the smallest shift), with collinear shifted residuals r_k = zeta_k r
// ---------------------------------------------------------------------------
constexpr int kMaxShifts = 16;
// The states an iteration reads (cur) and leaves behind (next): two sets, so that no workgroup of the
// launch that ends an iteration reads what another one writes.
struct MsSet {
    // per column
    double* rho;       // |r|^2
    double* alpha_prev;
    double* beta_prev;
    int* status;       // COL_ACTIVE / COL_DONE / COL_FAILED
    int* iters;
    // per column and shift, index c * nshift + k
    double* zeta;      // zeta_j
    double* zeta_prev; // zeta_{j-1}
    int* act;          // shift still iterating
    int* kiters;       // iterations of the shift
};
struct MsState {
    MsSet cur, next;
    double* alpha;     // per column: base alpha_j
    double* stop2;     // (tol |b|)^2
    double* zeta_new;  // per column and shift: zeta_{j+1}
    double* ak;        // shift alpha
    int nshift, base;
    double shift[kMaxShifts];  // sigma_k - sigma_b
};
struct MsFields {
    FieldArg r, w, p;              // base residual, A p (without the base shift), base direction
    FieldArg x[kMaxShifts];        // solutions
    FieldArg pk[kMaxShifts];       // shift directions (pk[base] = p)
};
hipError_t launch_ms_init(const MsState& s, int ncol, double tol2, hipStream_t st);
// alpha of the base system from the nparts partials of |q|^2 (and |p|^2 if sigma_b), zeta_{j+1} and alpha of
// the shifts; r -= alpha (w + sigma_b p); |r|^2 partials
hipError_t launch_ms_residual(const MsState& s, const MsFields& f, const double* pq, const double* pp, int nparts,
                              double sigma_b, int n, int ncol, double* partial, int nwaves, hipStream_t st);
// beta from the nparts partials of |r|^2; per active shift x_k += ak p_k, then p_k = zeta_{j+1} r + bk p_k (base:
// p = r + beta p) unless it has converged; |p|^2 partials; the states after the iteration into s.next
hipError_t launch_ms_directions(const MsState& s, const MsFields& f, const double* pr, int nparts, int n, int ncol,
                                double* partial, int nwaves, hipStream_t st);

// ---------------------------------------------------------------------------
// block (multishift) CG: one block Krylov space for N <= kBlockMax columns; the N x N step
// matrices live on the device and are computed there by one wavefront, so a run needs no host
// round trip per iteration
// ---------------------------------------------------------------------------
constexpr int kBlockMax = 16;   // columns of a block solve
// control words
enum { BC_K = 0, BC_STOP = 1, BC_BREAK = 2, BC_NA = 3, BC_MASK = 4, BC_IDX = 5,
       BC_FROZEN = BC_IDX + kBlockMax, BC_COUNT = BC_FROZEN + kMaxShifts };
// matrix slots (kBlockMax x kBlockMax complex each, row-major).  "Full" matrices are indexed by
// column number and vanish outside the active columns; "packed" ones hold the na x na block of the
// active columns in the order of the active list.
enum { BM_PQ = 0,       // full: P^dag (A P + sigma_b P)
       BM_RR = 1,       // full: R^dag R of the current residual block
       BM_RRN = 2,      // full: R^dag R of the new residual block
       BM_ALPHA = 3,    // full: base step matrix alpha_k
       BM_BETA = 4,     // full: base direction matrix beta_k
       BM_AINV = 5,     // packed: alpha_k^-1
       BM_C = 6,        // packed: alpha_k^-1 beta_k
       BM_SHIFT = 7 };  // per shift s at BM_SHIFT + 6 s: packed xi_k, packed xi_k-1, packed alpha^s_k-1,
                        // full xi_k (for the direction update), full alpha^s_k, full beta^s_k-1
constexpr int kBlockMats = BM_SHIFT + 6 * kMaxShifts;
struct BlockState {
    double2* mats;   // kBlockMats matrices
    double* thr;     // per column: (tol |b_c|)^2
    int* ctrl;       // BC_* words
    int* colstat;    // per column: COL_ACTIVE while in the block, COL_DONE otherwise (stencil filter)
    int* sstat;      // per shift and column [s * ncol + c]: 0 iterating, 1 converged
    int* siters;     // per shift and column: iteration at which it converged
    int ncol, nshift, base;
    double sigma_b;                // shift of the base system (added to A P)
    double shift[kMaxShifts];      // sigma_s - sigma_b
};
struct BlockFields {
    FieldArg x[kMaxShifts];        // solutions (x[base] is the base iterate)
    FieldArg p[kMaxShifts];        // directions (p[base] is the base direction)
};
// partial Gram sums of <X_i, Y_j + s X_j> over the active columns (s = 0 where Y is X): per workgroup
// (block_gram_parts of them) one complex number per entry of a kBlockMax^2 matrix
int block_gram_parts(int tiles);
hipError_t launch_block_gram(FieldArg X, FieldArg Y, double s, const BlockState& S, int vh, int tiles, double2* partial,
                             hipStream_t st);
// fixed-order sum of the partials into matrix slot `slot` (full)
hipError_t launch_block_gram_fin(const BlockState& S, const double2* partial, int tiles, int slot, hipStream_t st);
// 0: start of a run (active list from colstat and the Gram matrix in BM_RR, dependent columns
// dropped); 1: alpha and the shift recurrences (after BM_PQ); 2: convergence, beta (after BM_RRN)
hipError_t launch_block_step(const BlockState& S, int phase, hipStream_t st);
// x_base += P alpha, R -= (W + sigma_b P) alpha
hipError_t launch_block_xr(const BlockState& S, FieldArg x, FieldArg p, FieldArg w, FieldArg r, size_t units,
                           hipStream_t st);
// P = R + P beta
hipError_t launch_block_p(const BlockState& S, FieldArg p, FieldArg r, size_t units, hipStream_t st);
// every shift s other than the base: p_s = R xi + p_s beta_s, x_s += p_s alpha_s
hipError_t launch_block_shift(const BlockState& S, const BlockFields& f, FieldArg r, size_t units, hipStream_t st);

// ---------------------------------------------------------------------------
// BiCGstab on Mhat (inner precision FP64 or FP32, FP64 reductions, FP64 restarts)
// ---------------------------------------------------------------------------
struct BicgScalars {
    double2* rho;     // <rhat, r>
    double2* alpha;
    double2* omega;
    double2* beta;
    double* r2;       // |r|^2 of the inner iteration
    double* stop2;    // inner goal |r|^2
    double* tol2b2;   // (tol |b|)^2 of the FP64 system
    double delta2;    // inner goal relative to the last FP64 residual
    int* status;      // COL_ACTIVE, COL_STOPPED (inner goal reached), COL_DONE, COL_FAILED
    int* iters;
    int* nrel;        // FP64 residual recomputations
    int* restart;     // set by the reliable pass for columns that restart
};
hipError_t launch_bicg_p(int prec, FieldArg r, FieldArg p, FieldArg v, const BicgScalars& s, int n, int ncol,
                         hipStream_t st);
// partials of <a1, b1> and (a2.d != null) <a2, b2>, [col][re1, im1, re2, im2][wave]
hipError_t launch_dots2(int prec, FieldArg a1, FieldArg b1, FieldArg a2, FieldArg b2, const int* status, int n,
                        int ncol, double* partial, int nwaves, hipStream_t st);
hipError_t launch_bicg_s(int prec, FieldArg r, FieldArg v, FieldArg s_, const BicgScalars& s, int n, int ncol,
                         hipStream_t st);
hipError_t launch_bicg_xr(int prec, FieldArg x, FieldArg p, FieldArg s_, FieldArg t, FieldArg r, FieldArg rhat,
                          const BicgScalars& s, int n, int ncol, double* partial, int nwaves, hipStream_t st);
// step 0: alpha, 1: omega, 2: rho / beta / stop test, 3: reliable pass decision (partials of |r64|^2)
hipError_t launch_fin_bicg(int step, const BicgScalars& s, const double* partial, int nwaves, int ncol,
                           hipStream_t st);

// CG finalisation kernels (one block per column)
struct CgScalars {
    double* rho;      // |r|^2 of the current iterate
    double* pAp;
    double* alpha;
    double* beta;
    double* stop2;    // (tol * |b|)^2
    double* rmax2;    // reliable-update reference |r|^2 (delta test)
    double delta2;    // delta^2 (0 = no reliable trigger)
    int* status;
    int* iters;
    int* restart;
    int* nrel;        // reliable updates per column
};
// launch_fin_beta and launch_cg_update in one, for up to kFusedParts partials per column, after a stencil that
// took alpha itself: every workgroup takes its column's sum itself; the states after the iteration
// go to `next` (its rho, rmax2, status and iters; for every column), also those that launch_fin_alpha would set
constexpr int kFusedParts = 1024;
hipError_t launch_cg_update_beta(int xprec, FieldArg x, int pprec, FieldArg p, int rprec, FieldArg r, int n, int ncol,
                                 const CgScalars& cur, const CgScalars& next, const double* partial, int nwaves,
                                 hipStream_t st);
hipError_t launch_fin_alpha(const CgScalars& s, const double* partial, int nwaves, int ncol, hipStream_t st);
hipError_t launch_fin_beta(const CgScalars& s, const double* partial, int nwaves, int ncol, hipStream_t st);
hipError_t launch_fin_reliable(const CgScalars& s, const double* partial, int nwaves, int ncol, hipStream_t st);
hipError_t launch_fin_max(const double* partial, int n, double* out, hipStream_t st);  // the largest of n
hipError_t launch_fin_sum(const double* partial, int nwaves, int ncol, double* out, hipStream_t st);
// stop2 = tol2 * rho, rmax2 = rho, counters cleared, status from rho (rho holds |b|^2 on entry);
// with `sel` only columns with sel[c] != 0 are initialised, and tol2 is per column (tol2c) if given
hipError_t launch_cg_init(const CgScalars& s, int ncol, double tol2, hipStream_t st, const int* sel = nullptr,
                          const double* tol2c = nullptr, const double* rho_src = nullptr);
// status[c] = value for every column with sel[c] != 0
hipError_t launch_set_status(int* status, const int* sel, int ncol, int value, hipStream_t st);

}  // namespace bq
